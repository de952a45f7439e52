// gfx950 kernels of the X-engine correlator.
//
// The hot kernel (xcorr_mfma) computes, for one 128 x 128 tile (ti, tj) of
// the upper triangle and one range of time samples, the visibilities
//   V_ij = sum_t x_i(t) conj(x_j(t))                      (Sec. 2.2, eta)
// of 4+4-bit offset-encoded samples and adds them into int32 accumulators.
//
// The complex product is split into two real int8 contractions over a
// K axis that carries the real parts of a k-step's 16 samples on MFMA lanes
// 0-31 and the imaginary parts on lanes 32-63:
//   Re V = [Re x_i | Im x_i] . [Re x_j | Im x_j]    = Re_i Re_j + Im_i Im_j
//   Im'  = [Im x_i | ~Re x_i] . [Re x_j | Im x_j]   = Im_i Re_j - Re_i Im_j - Im_j
// with ~Re = -Re - 1 (the bitwise complement of the 4-bit value, which,
// unlike -Re, never leaves [-8, 7]).  So the row (A) side keeps three int8
// vectors per sample group (Re, Im, ~Re) and the column (B) side two (Re,
// Im); one B operand feeds both products.  The stored imaginary part is
// Im V_ij - S_j with S_j = sum_t Im x_j(t); as Im V_jj = 0, the diagonal
// holds -S_j, which also goes to the slot's biases, and the dump adds S_j
// back.  Every partial sum is an exact int32.  The DMA kernel stores the same
// form.
//
// Data path per 32-sample stage (double-buffered in LDS):
//   global (time-major bytes) -> dword loads, 4 inputs x 8 samples per lane
//   -> 4x4 byte transposes (v_perm) -> nibble unpack to int8 -> LDS
//   -> ds_read_b128 operands -> v_mfma_i32_32x32x32_i8.
// The paper's own design packed several low-bit products into 24-bit
// multiply-adds on GCN3 (Sec. 2.3, "GPUs"); on CDNA4 the int8 matrix cores
// do this work instead (Sec. 4.1 anticipates low-bit matrix units).
//
// FP8 instances (an exact matrix-core path on 8-bit floats, Sec. 4.1's
// low-bit matrix units) stage every 4-bit value v in [-8, 7] as its OCP
// E4M3 code (1 sign, 4 exponent bits with bias 7, 3 mantissa bits: every
// integer of magnitude <= 16 is exact, -v included, so the imaginary
// operand is [Im | -Re] and carries no bias) and multiply on
// v_mfma_f32_32x32x16_fp8_fp8 into fp32 accumulators.  Products are
// exact, and fp32 sums of integers are exact while below 2^24: with at most
// 128 per sample, pieces below 2^17 samples flush exact integers, converted
// to int32.
//
// UNSIGNED instances multiply the stored nibbles u = x + 8 themselves (the
// paper's unsigned form, whose O(N) bookkeeping is the pre-sum correction
// of xeng_presum.hip): A = [uR | uI] and [uI | -uR], B = [8 uR | 8 uI], so
// the sums are 8 x sum (uR_i uR_j + uI_i uI_j) and 8 x sum (uI_i uR_j -
// uR_i uI_j), flushed with a shift of 3.  At most 3600 per sample, so such
// pieces stay below 2^19 samples (int32 register sums).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "xeng_internal.h"

namespace xeng {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// LDS stage layout.  A stage is 64 samples = 4 MFMA k-steps.  For each
// k-step q a component region holds 128 tile rows x 16 bytes (the 16
// samples of one input, in time order).  A rows keep Re, Im, ~Re as int8;
// B rows keep 16*Re, 16*Im as int8 (the scale makes their unpack three bit
// operations per four samples; every product is then 16x the true one and
// the flush divides it out exactly).  This is the general kernel, for any
// alignment and N; 16-byte-aligned arrays take the DMA kernel instead.
constexpr int CH = TILE * 16;       // 2048 bytes
constexpr int QSTEPS = STAGE / KSTEP;   // 4
constexpr int A_Q = 3 * CH;
constexpr int B_Q = 2 * CH;
constexpr int A_BYTES = QSTEPS * A_Q;   // 24 KB
constexpr int B_BYTES = QSTEPS * B_Q;   // 16 KB
constexpr int STAGE_BYTES = A_BYTES + B_BYTES;   // 40 KB
constexpr int NBUF = 2;

__device__ __forceinline__ uint32_t vperm(uint32_t s0, uint32_t s1, uint32_t sel)
{
    return __builtin_amdgcn_perm(s0, s1, sel);
}

// 4 x 4 byte transpose: in[t] holds 4 inputs at time t; out[c] holds input
// c at the 4 times (byte = time).
__device__ __forceinline__ void transpose4(uint32_t i0, uint32_t i1, uint32_t i2, uint32_t i3,
                                           uint32_t &o0, uint32_t &o1, uint32_t &o2, uint32_t &o3)
{
    const uint32_t ab_lo = vperm(i1, i0, 0x05010400u);   // a0 b0 a1 b1
    const uint32_t ab_hi = vperm(i1, i0, 0x07030602u);   // a2 b2 a3 b3
    const uint32_t cd_lo = vperm(i3, i2, 0x05010400u);
    const uint32_t cd_hi = vperm(i3, i2, 0x07030602u);
    o0 = vperm(cd_lo, ab_lo, 0x05040100u);               // a0 b0 c0 d0
    o1 = vperm(cd_lo, ab_lo, 0x07060302u);               // a1 b1 c1 d1
    o2 = vperm(cd_hi, ab_hi, 0x05040100u);
    o3 = vperm(cd_hi, ab_hi, 0x07060302u);
}

// Offset-binary nibbles (0..15, one per byte) -> signed int8 value v = n - 8
// and its complement ~v = -v - 1 = 7 - n, four at a time, with no carries
// between bytes:
//   n - 8 = (n + 0x78) ^ 0x80,   7 - n = (0x87 - n) ^ 0x80.
__device__ __forceinline__ uint32_t nib_to_i8(uint32_t n) { return (n + 0x78787878u) ^ 0x80808080u; }
__device__ __forceinline__ uint32_t nib_to_not_i8(uint32_t n) { return (0x87878787u - n) ^ 0x80808080u; }

// Offset-binary nibbles (0..15, one per byte) -> the E4M3 codes of v = n - 8,
// four at a time.  For n >= 8 the code of v = n - 8 in 0..7 is
// POS[n - 8]; for n < 8, v = -(8 - n) and the code is 0x80 | NEG[n] with
// NEG[n] the code of 8 - n.  Codes: 1 = 0x38 (2^0), 2 = 0x40, 3 = 0x44
// (1.5 x 2), 4 = 0x48, 5 = 0x4A (1.25 x 4), 6 = 0x4C, 7 = 0x4E, 8 = 0x50.
// Each table is eight bytes, read by a byte permute with selector n & 7;
// bit 3 of n picks the table.
constexpr uint32_t E4M3_POS_LO = 0x44403800u, E4M3_POS_HI = 0x4E4C4A48u;   // v = 0, 1, .. 7
constexpr uint32_t E4M3_NEG_LO = 0x4A4C4E50u, E4M3_NEG_HI = 0x38404448u;   // |v| = 8, 7, .. 1
__device__ __forceinline__ uint32_t nib_to_e4m3(uint32_t n)
{
    const uint32_t sel = n & 0x07070707u;
    const uint32_t pos = vperm(E4M3_POS_HI, E4M3_POS_LO, sel);
    const uint32_t neg = vperm(E4M3_NEG_HI, E4M3_NEG_LO, sel) | 0x80808080u;
    const uint32_t hi = ((n >> 3) & 0x01010101u) * 0xFFu;   // 0xFF in the bytes with n >= 8
    return (pos & hi) | (neg & ~hi);
}

// Global-memory views: loads through these pointers are global (not flat)
// instructions, so they only count against the vector-memory counter and
// stay in flight while the LDS reads and MFMAs of the current stage run.
typedef __attribute__((address_space(1))) const u32x2 gcu64;
typedef __attribute__((address_space(1))) const uint8_t gcu8;
// the same eight bytes at any byte address
typedef u32x2 u32x2_u __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) const u32x2_u gcu64u;
typedef __attribute__((address_space(1))) uint64_t gw64;

// One lane's share of a stage: 8 inputs x 8 consecutive samples of one
// block (d[k] = the 8 inputs at sample k), as loaded, plus a mask of which
// samples are real (bit k) -- the others become the zero sample at unpack.
struct StageRegs {
    u32x2 d[8];
    uint32_t valid;
};
constexpr uint32_t ALL_VALID = 0xFFu;

// Per-piece constants of one lane.
struct PieceCtx {
    const uint8_t *samples;
    int64_t stride;
    int n, t0, t1;
    int i0;               // first of the 8 inputs this lane stages
    uint32_t off;         // lane byte offset from a stage's first time row
    bool full_rows;       // all 128 inputs of this lane's block are < n
    int t_lane;           // first sample of this lane inside a stage
};

// Fast stage: every sample and input in range.  Eight 8-byte loads at a
// uniform row base plus a 32-bit lane offset.
__device__ __forceinline__ void load_fast(StageRegs &r, const uint8_t *row0, int64_t stride,
                                          uint32_t off)
{
#pragma unroll
    for (int k = 0; k < 8; ++k) r.d[k] = *(gcu64 *)(row0 + (int64_t)k * stride + off);
    r.valid = ALL_VALID;
}

// Edge stage: the same eight loads with every address clamped into the
// array.  Nothing loaded is consumed here, so the loads of both paths stay
// in flight and the memory-counter waits stay precise.
__device__ __forceinline__ void load_clamped(StageRegs &r, const PieceCtx &pc, int t_first)
{
    const bool vi = pc.i0 < pc.n;
    uint32_t valid = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int t = t_first + k;
        const bool vt = t < pc.t1;
        const uint8_t *row = pc.samples + (int64_t)(vt ? t : pc.t0) * pc.stride;
        r.d[k] = *(gcu64 *)(row + (vi ? pc.i0 : 0));
        valid |= ((vt && vi) ? 1u : 0u) << k;
    }
    r.valid = valid;
}

// Unaligned rows (a base or stride not a multiple of 8, or N not a multiple
// of 8): one 8-byte load per row at any byte address -- global loads run in
// unaligned-access mode, which the compiler also assumes for align-1 loads.
// A lane whose eight inputs cross input N - 1 reads the eight bytes that end
// there and shifts its own down to the bottom, so no load reaches past the
// row's N bytes; the inputs past N become the zero sample.  For N < 8 the
// one lane with inputs reads them byte by byte.
__device__ __forceinline__ void load_unaligned(StageRegs &r, const PieceCtx &pc, int t_first)
{
    constexpr uint64_t ZERO8 = 0x8888888888888888ull;
    const int nb = pc.n - pc.i0;                                  // this lane's inputs that exist
    const int off = min(pc.i0, pc.n - 8);                         // first byte read (n >= 8)
    const uint32_t sh = 8u * (uint32_t)(pc.i0 - off);             // bits below this lane's first input
    const uint64_t keep = nb >= 8 ? ~0ull : nb > 0 ? (1ull << (8 * nb)) - 1 : 0ull;
    uint32_t valid = 0;
    if (pc.n >= 8) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t = t_first + k;
            const bool vt = t < pc.t1;
            const uint8_t *row = pc.samples + (int64_t)(vt ? t : pc.t0) * pc.stride;
            uint64_t v = ZERO8;
            if (nb > 0) {
                const u32x2 w = *(gcu64u *)(row + off);
                v = ((((uint64_t)w.y << 32) | w.x) >> sh & keep) | (ZERO8 & ~keep);
            }
            r.d[k] = u32x2{(uint32_t)v, (uint32_t)(v >> 32)};
            valid |= (vt ? 1u : 0u) << k;
        }
    } else {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int t = t_first + k;
            const bool vt = t < pc.t1;
            const uint8_t *row = pc.samples + (int64_t)(vt ? t : pc.t0) * pc.stride;
            uint64_t v = ZERO8;
            for (int b = 0; b < nb; ++b)
                v = (v & ~(0xFFull << (8 * b))) | ((uint64_t)((gcu8 *)row)[pc.i0 + b] << (8 * b));
            r.d[k] = u32x2{(uint32_t)v, (uint32_t)(v >> 32)};
            valid |= (vt ? 1u : 0u) << k;
        }
    }
    r.valid = valid;
}

template <bool ALIGNED>
__device__ __forceinline__ void load_stage(StageRegs &r, const PieceCtx &pc, int s)
{
    const int ts = pc.t0 + s * STAGE;
    if (!ALIGNED)
        load_unaligned(r, pc, ts + pc.t_lane);
    else if (pc.full_rows && ts + STAGE <= pc.t1)
        load_fast(r, pc.samples + (int64_t)ts * pc.stride, pc.stride, pc.off);
    else
        load_clamped(r, pc, ts + pc.t_lane);
}

// Unpack one lane's share of a stage into the stage buffer.  `slot` is the
// byte offset of this lane's (first input, half) in a component region;
// input c of the lane sits 16 * c bytes further.
template <bool ROLE_A, bool RE_LOW, bool UNSIGNED, bool FP8>
__device__ __forceinline__ void stage_write(uint8_t *region, const StageRegs &r, int slot)
{
    uint32_t lo[8], hi[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        lo[k] = r.d[k].x;
        hi[k] = r.d[k].y;
    }
    if (r.valid != ALL_VALID) {     // uniform in the steady state
        // samples past the piece's end (or past N) become the zero sample;
        // in the unsigned form the zero sample u = 8 would add 64 per
        // product, so there they become u = 0, which adds nothing
        const uint32_t fill = UNSIGNED ? 0u : 0x88888888u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool ok = (r.valid >> k) & 1u;
            lo[k] = ok ? lo[k] : fill;
            hi[k] = ok ? hi[k] : fill;
        }
    }
    // p[c][h]: input c, samples 4h..4h+3
    uint32_t p[8][2];
    transpose4(lo[0], lo[1], lo[2], lo[3], p[0][0], p[1][0], p[2][0], p[3][0]);
    transpose4(lo[4], lo[5], lo[6], lo[7], p[0][1], p[1][1], p[2][1], p[3][1]);
    transpose4(hi[0], hi[1], hi[2], hi[3], p[4][0], p[5][0], p[6][0], p[7][0]);
    transpose4(hi[4], hi[5], hi[6], hi[7], p[4][1], p[5][1], p[6][1], p[7][1]);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        uint8_t *dst = region + slot + 16 * c;
        if (UNSIGNED) {
            // the stored nibbles u in 0..15, no offset removed: A rows keep
            // uR, uI and -uR (per byte (0x80 - u) ^ 0x80, no borrows); B
            // rows 8 uR, 8 uI (at most 120: int8)
            const uint32_t h0 = (p[c][0] >> 4) & 0x0F0F0F0Fu, l0 = p[c][0] & 0x0F0F0F0Fu;
            const uint32_t h1 = (p[c][1] >> 4) & 0x0F0F0F0Fu, l1 = p[c][1] & 0x0F0F0F0Fu;
            const uint32_t re0 = RE_LOW ? l0 : h0, im0 = RE_LOW ? h0 : l0;
            const uint32_t re1 = RE_LOW ? l1 : h1, im1 = RE_LOW ? h1 : l1;
            if (ROLE_A) {
                *(uint2 *)(dst) = make_uint2(re0, re1);
                *(uint2 *)(dst + CH) = make_uint2(im0, im1);
                *(uint2 *)(dst + 2 * CH) =
                    make_uint2((0x80808080u - re0) ^ 0x80808080u, (0x80808080u - re1) ^ 0x80808080u);
            } else {
                *(uint2 *)(dst) = make_uint2(re0 << 3, re1 << 3);
                *(uint2 *)(dst + CH) = make_uint2(im0 << 3, im1 << 3);
            }
            continue;
        }
        if (FP8) {
            // A rows: Re, Im, -Re; B rows: Re, Im (E4M3 codes; -v flips
            // the sign bit, exactly)
            const uint32_t h0 = (p[c][0] >> 4) & 0x0F0F0F0Fu, l0 = p[c][0] & 0x0F0F0F0Fu;
            const uint32_t h1 = (p[c][1] >> 4) & 0x0F0F0F0Fu, l1 = p[c][1] & 0x0F0F0F0Fu;
            const uint32_t re0 = nib_to_e4m3(RE_LOW ? l0 : h0), im0 = nib_to_e4m3(RE_LOW ? h0 : l0);
            const uint32_t re1 = nib_to_e4m3(RE_LOW ? l1 : h1), im1 = nib_to_e4m3(RE_LOW ? h1 : l1);
            *(uint2 *)(dst) = make_uint2(re0, re1);
            *(uint2 *)(dst + CH) = make_uint2(im0, im1);
            if (ROLE_A) *(uint2 *)(dst + 2 * CH) = make_uint2(re0 ^ 0x80808080u, re1 ^ 0x80808080u);
            continue;
        }
        if (ROLE_A) {
            const uint32_t h0 = (p[c][0] >> 4) & 0x0F0F0F0Fu, l0 = p[c][0] & 0x0F0F0F0Fu;
            const uint32_t h1 = (p[c][1] >> 4) & 0x0F0F0F0Fu, l1 = p[c][1] & 0x0F0F0F0Fu;
            const uint32_t re0 = RE_LOW ? l0 : h0, im0 = RE_LOW ? h0 : l0;
            const uint32_t re1 = RE_LOW ? l1 : h1, im1 = RE_LOW ? h1 : l1;
            *(uint2 *)(dst) = make_uint2(nib_to_i8(re0), nib_to_i8(re1));
            *(uint2 *)(dst + CH) = make_uint2(nib_to_i8(im0), nib_to_i8(im1));
            *(uint2 *)(dst + 2 * CH) = make_uint2(nib_to_not_i8(re0), nib_to_not_i8(re1));
        } else {
            // flipping bit 3 of an offset-binary nibble gives its 4-bit two's
            // complement; in the high half of a byte that is 16x the value
            const uint32_t x0 = p[c][0] ^ 0x88888888u, x1 = p[c][1] ^ 0x88888888u;
            const uint32_t xh0 = x0 & 0xF0F0F0F0u, xl0 = (x0 << 4) & 0xF0F0F0F0u;
            const uint32_t xh1 = x1 & 0xF0F0F0F0u, xl1 = (x1 << 4) & 0xF0F0F0F0u;
            *(uint2 *)(dst) = RE_LOW ? make_uint2(xl0, xl1) : make_uint2(xh0, xh1);
            *(uint2 *)(dst + CH) = RE_LOW ? make_uint2(xh0, xh1) : make_uint2(xl0, xl1);
        }
    }
}

__device__ __forceinline__ v4i lds128(const uint8_t *p) { return *(const v4i *)p; }

// An accumulator register as the integer it holds (fp32 sums of the FP8
// instances are exact integers below 2^24).
__device__ __forceinline__ int32_t acc_int(int32_t v) { return v; }
__device__ __forceinline__ int32_t acc_int(float v) { return (int32_t)v; }

// Accumulators hold 16x the stored values (B operands are scaled by 16), so
// the flush adds acc >> 4; every value is a multiple of 16, so this is
// exact.  Pairs go to the slot as packed 64-bit words (see the layout note):
// a shared tile takes one 64-bit atomic add per pair.
template <int SHIFT, typename V>
__device__ __forceinline__ void flush_block(gw64 *blk, const V &re, const V &im)
{
#pragma unroll
    for (int r = 0; r < 16; ++r)
        __hip_atomic_fetch_add(blk + r * 64, pack_pair(acc_int(re[r]) >> SHIFT, acc_int(im[r]) >> SHIFT),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool FP8> struct AccT {
    v16i re[2][2];
    v16i im[2][2];
};
template <> struct AccT<true> {
    v16f re[2][2];
    v16f im[2][2];
};
typedef AccT<false> Acc;


// Whole-tile flush of one wave's 2 x 2 blocks: stores if the slot holds
// zeros, else read-modify-write with the loads of a row of blocks issued
// before their stores (one memory latency per row, not one per value).
template <int SHIFT, bool FP8>
__device__ __forceinline__ void flush_owned(gw64 *tb, const AccT<FP8> &acc, int wa, int wb, bool fresh)
{
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        gw64 *blk[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) blk[b] = tb + ((2 * wa + a) * BLKS + (2 * wb + b)) * BLOCK_W;
        uint64_t old[2][16];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) old[b][r] = fresh ? 0 : blk[b][r * 64];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                blk[b][r * 64] =
                    old[b][r] + pack_pair(acc_int(acc.re[a][b][r]) >> SHIFT, acc_int(acc.im[a][b][r]) >> SHIFT);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The FP8 form of a k-step's products: each 16-byte operand is two 8-byte
// E4M3 operands of v_mfma_f32_32x32x16_fp8_fp8 (samples 0..7 of the
// k-step's Re and Im halves, then samples 8..15).
__device__ __forceinline__ v16f mfma_fp8(const v4i &a, const v4i &b, v16f c)
{
    const long a0 = (long)(((uint64_t)(uint32_t)a.y << 32) | (uint32_t)a.x);
    const long a1 = (long)(((uint64_t)(uint32_t)a.w << 32) | (uint32_t)a.z);
    const long b0 = (long)(((uint64_t)(uint32_t)b.y << 32) | (uint32_t)b.x);
    const long b1 = (long)(((uint64_t)(uint32_t)b.w << 32) | (uint32_t)b.z);
    c = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a0, b0, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(a1, b1, c, 0, 0, 0);
}

__device__ __forceinline__ v16i mfma_k(const v4i &a, const v4i &b, v16i c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v16f mfma_k(const v4i &a, const v4i &b, v16f c) { return mfma_fp8(a, b, c); }

// The 32 MFMAs of one stage (4 k-steps x 2 x 2 blocks x Re/Im) on `buf`
// (64 for the FP8 instances, two per block and k-step).
template <bool FP8>
__device__ __forceinline__ void stage_mfma(AccT<FP8> &acc, const uint8_t *buf, int lane, int wa, int wb)
{
#pragma unroll
    for (int q = 0; q < QSTEPS; ++q) {
        const uint8_t *aq = buf + q * A_Q + (lane >> 5) * CH + 16 * (lane & 31);
        const v4i re_a0 = lds128(aq + 512 * (2 * wa));
        const v4i re_a1 = lds128(aq + 512 * (2 * wa + 1));
        const v4i im_a0 = lds128(aq + CH + 512 * (2 * wa));
        const v4i im_a1 = lds128(aq + CH + 512 * (2 * wa + 1));
        const uint8_t *bp = buf + A_BYTES + q * B_Q + (lane >> 5) * CH + 16 * (lane & 31);
        const v4i b0 = lds128(bp + 512 * (2 * wb));
        const v4i b1 = lds128(bp + 512 * (2 * wb + 1));
        acc.re[0][0] = mfma_k(re_a0, b0, acc.re[0][0]);
        acc.im[0][0] = mfma_k(im_a0, b0, acc.im[0][0]);
        acc.re[0][1] = mfma_k(re_a0, b1, acc.re[0][1]);
        acc.im[0][1] = mfma_k(im_a0, b1, acc.im[0][1]);
        acc.re[1][0] = mfma_k(re_a1, b0, acc.re[1][0]);
        acc.im[1][0] = mfma_k(im_a1, b0, acc.im[1][0]);
        acc.re[1][1] = mfma_k(re_a1, b1, acc.re[1][1]);
        acc.im[1][1] = mfma_k(im_a1, b1, acc.im[1][1]);
    }
}

// Correlate one piece: tile (ti, tj) over samples [t0, t1).  Stage s is in
// LDS being multiplied while stage s+1 (in registers) is unpacked into the
// other LDS buffer and stage s+2 loads from memory.  Steps run in pairs with
// no early exit: a stage past the end of the piece holds zero samples and
// adds exactly nothing.
template <bool ALIGNED, bool ROLE_A, bool RE_LOW, bool UNSIGNED, bool FP8>
__device__ __forceinline__ void run_piece(AccT<FP8> &acc, uint8_t *smem, const PieceCtx &pc, int lane,
                                          int wa, int wb, int wslot, bool compute)
{
    const int nst = (pc.t1 - pc.t0 + STAGE - 1) / STAGE;
    uint8_t *buf0 = smem, *buf1 = smem + STAGE_BYTES;
    StageRegs r0, r1;

    load_stage<ALIGNED>(r0, pc, 0);
    load_stage<ALIGNED>(r1, pc, 1);
    stage_write<ROLE_A, RE_LOW, UNSIGNED, FP8>(buf0, r0, wslot);
    __syncthreads();

    for (int s = 0; s < nst; s += NBUF) {
        load_stage<ALIGNED>(r0, pc, s + 2);
        if (compute) stage_mfma<FP8>(acc, buf0, lane, wa, wb);
        stage_write<ROLE_A, RE_LOW, UNSIGNED, FP8>(buf1, r1, wslot);
        __syncthreads();
        load_stage<ALIGNED>(r1, pc, s + 3);
        if (compute) stage_mfma<FP8>(acc, buf1, lane, wa, wb);
        stage_write<ROLE_A, RE_LOW, UNSIGNED, FP8>(buf0, r0, wslot);
        __syncthreads();
    }
}

// Persistent correlation kernel: workgroup w runs pieces [wg_off[w], wg_off[w+1]).
// 256 threads = 4 waves; wave (wa, wb) owns MFMA blocks ca in {2wa, 2wa+1},
// cb in {2wb, 2wb+1} of the tile (64 x 64 outputs, Re and Im).  Staging:
// waves 0-1 unpack the A (row) block, waves 2-3 the B (column) block; a lane
// takes 8 inputs x 8 samples (lane bits 0-2 and 4 pick the 8-input group,
// bit 3 the half of a k-step, bit 5 and the wave the k-step).
template <bool ALIGNED, bool UNSIGNED, bool FP8>
__global__ __launch_bounds__(256, 2) void xcorr_mfma(KernelArgs args)
{
    __shared__ __attribute__((aligned(16))) uint8_t smem[NBUF * STAGE_BYTES];
    // a prepared batch's device guard refused this launch
    if (args.skip != nullptr && *args.skip != 0) return;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wa = wave >> 1, wb = wave & 1;
    const bool role_a = wave < 2;
    const int g8 = (lane & 7) | (((lane >> 4) & 1) << 3);   // 8-input group 0..15
    const int half = (lane >> 3) & 1;                        // samples 0-7 / 8-15 of a k-step
    const int q = 2 * (wave & 1) + (lane >> 5);              // k-step 0..3
    // LDS byte offset of this lane's (input 8*g8, half, k-step); input c of
    // the lane is 16 * c bytes further
    const int wslot = (role_a ? q * A_Q : A_BYTES + q * B_Q) + 128 * g8 + 8 * half;

    const int p_begin = args.wg_off[blockIdx.x], p_end = args.wg_off[blockIdx.x + 1];
    for (int pi = p_begin; pi < p_end; ++pi) {
        const Piece pce = args.pieces[pi];
        const JobDesc jd = args.jobs ? args.jobs[pce.job] : args.job0;
        const int ti = pce.tile & 0xFFFF, tj = (pce.tile >> 16) & 0xFFFF;
        const bool atomic = pce.t1_atomic < 0;
        const int blk0 = (role_a ? ti : tj) * TILE;

        PieceCtx pc;
        pc.samples = jd.samples;
        pc.stride = jd.stride;
        pc.n = jd.n;
        pc.t0 = pce.t0;
        pc.t1 = pce.t1_atomic & 0x7FFFFFFF;
        pc.i0 = blk0 + 8 * g8;
        pc.t_lane = 16 * q + 8 * half;
        // lane offset from a stage's first row: fits 32 bits (stride <= 2^26)
        pc.off = (uint32_t)(pc.t_lane * jd.stride) + (uint32_t)pc.i0;
        pc.full_rows = blk0 + TILE <= jd.n;

        AccT<FP8> acc;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc.re[a][b][r] = 0;
                    acc.im[a][b][r] = 0;
                }

        const bool re_low = (jd.flags & JOB_RE_LOW) != 0;
        // a wave whose 64 x 64 region lies wholly past the last input (rows
        // or columns >= N) or below the diagonal is never exported: it stages
        // its share but multiplies and flushes nothing (a diagonal tile's
        // words down there hold the slot's bias bases, see BASE_I32)
        const bool compute = TILE * ti + 64 * wa < jd.n && TILE * tj + 64 * wb < jd.n && !(ti == tj && wa > wb);
        if (role_a) {
            if (re_low) run_piece<ALIGNED, true, true, UNSIGNED, FP8>(acc, smem, pc, lane, wa, wb, wslot, compute);
            else run_piece<ALIGNED, true, false, UNSIGNED, FP8>(acc, smem, pc, lane, wa, wb, wslot, compute);
        } else {
            if (re_low) run_piece<ALIGNED, false, true, UNSIGNED, FP8>(acc, smem, pc, lane, wa, wb, wslot, compute);
            else run_piece<ALIGNED, false, false, UNSIGNED, FP8>(acc, smem, pc, lane, wa, wb, wslot, compute);
        }

        // integrate into the slot's accumulators: the signed int8 sums carry
        // 16x the value, the unsigned 8x, the FP8 ones the value itself
        if (!compute) continue;
        constexpr int SHIFT = FP8 ? 0 : UNSIGNED ? 3 : 4;
        const int64_t tile_idx = (int64_t)ti * jd.nt - (int64_t)ti * (ti - 1) / 2 + (tj - ti);
        gw64 *tb = (gw64 *)(jd.acc + tile_idx * TILE_I32) + lane;
        // the diagonal's imaginary sums are the slot's biases (the FP8 and
        // unsigned instances carry none)
        if constexpr (!UNSIGNED && !FP8)
            if (ti == tj && wa == wb && jd.bias != nullptr) {
                const int dr = diag_reg(lane);
#pragma unroll
                for (int a = 0; a < 2; ++a) {
                    int32_t v = 0;
#pragma unroll
                    for (int r = 0; r < 16; ++r) v = dr == r ? acc.im[a][a][r] : v;
                    const int j = TILE * ti + 64 * wa + BLK * a + (lane & 31);
                    if (dr >= 0 && j < jd.n)
                        __hip_atomic_fetch_add(jd.bias + j, v >> SHIFT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        if (atomic) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    flush_block<SHIFT>(tb + ((2 * wa + a) * BLKS + (2 * wb + b)) * BLOCK_W, acc.re[a][b],
                                acc.im[a][b]);
        } else if (jd.flags & JOB_FRESH) {
            flush_owned<SHIFT, FP8>(tb, acc, wa, wb, true);
        } else {
            flush_owned<SHIFT, FP8>(tb, acc, wa, wb, false);
        }
    }
}

// Export of a slot: accumulators (tile layout) -> packed row-major upper
// triangle of (Re, Im), optionally clearing the slot in the same pass.
// Bound by memory: 8 bytes read and written per exported pair, and 8 more
// written where it clears.
//
// A workgroup takes DUMP_ROWS rows x 128 columns of a tile, a wave one row
// at a time: lane c takes the two consecutive words of columns
// 32 (c / 16) + 2 (c % 16) .. + 1, so a row is read as four coalesced
// 256-byte runs, and writes its two pairs straight to the output row, 1 KB
// contiguous per wave (16-byte stores at 8-byte alignment).  Rows r and
// r + 4 of an 8-row group lie next to each other in the accumulators; every
// load of a thread is issued before its first store.  Pairs of
// inputs at or past n and 32 x 32 blocks below the diagonal are neither read
// nor cleared: whatever their words hold is never exported.  The imaginary
// part of (i, j) is stored as Im V_ij - S_j, so bias[j] - base[j] = -S_j is
// subtracted (exact in wrapping int32 arithmetic, since Im V_ij itself fits).
//
// Measured: N = 2048 with reset 9.8 us = 5.4 TB/s (4 rows per workgroup 9.4,
// 16 9.8, 32 10.4); as two kernels, the diagonal gathered first, 4.8 + 9.1.
// 1024 slots of N = 64 in one launch 27 us (4 rows 36, 16 24), where reading
// and clearing every tile whole took 44 us + 4.5 for the diagonals; 64
// sub-arrays of N 256 to 2048 136 us, where a grid sized for the largest
// job's tiles took 202.
//
// PAST: what a resetting export does past the caches once its launch's
// accumulators outgrow them (see STREAM_BYTES): from there on the output
// (1), which would only push out the words that the next integration adds to;
// from DUMP_PAST_BYTES on its reads and clears too, four rows per workgroup
// (2).  us of one correlation of 1024 samples and the exports, form 0 / 1 / 2: 12
// slots of N = 2048 236 / 227 / 243, 32 581 / 576 / 602, 64 (1 GiB) 1136 / 1134
// / 1119; 8 of N = 4096 580 / 557 / 574.  The exports alone: 12 slots 120 / 80 /
// 113, 32 322 / 326 / 294, 64 649 / 653 / 592.  Below, form 0: 6 slots 44 / 61
// (2).  Exports that keep the sums: 64 slots 374 / 383 / 387.
constexpr int64_t DUMP_PAST_BYTES = 4 * STREAM_BYTES;
template <int PAST> constexpr int DUMP_ROWS = PAST == 2 ? 4 : 8;
constexpr int DUMP_WAVES = 4;
template <int PAST> constexpr int DUMP_PARTS = TILE / DUMP_ROWS<PAST>;   // workgroups per tile

// A pending unsigned-form correction (CORR; see presum_correct): per
// input, SR at sums[i] and SI at sums[n4 + i] over the t samples that form
// contributed.  It is added to each word in the packed 64-bit form, before
// the word is split into (Re, Im): the uncorrected real part may have passed
// the int32 range, which the split would carry into Im.  `other` (the
// slot's second pre-sum buffer, 2 n4 int32, which the next calls of that
// form will use) is cleared on the way.
struct PendingCorr {
    const int32_t *sums;
    int32_t *other;
    int n4;
    int64_t t;
};
__device__ __forceinline__ uint64_t corr_word(int64_t ri, int64_t ii, int64_t rj, int64_t ij, int64_t t)
{
    const int64_t d_re = -8 * (ri + ii + rj + ij) + 128 * t;
    const int64_t d_im = 8 * (ri - ii) - 8 * (rj - ij);
    return ((uint64_t)d_im << 32) + (uint64_t)d_re;
}

typedef int dv4i __attribute__((ext_vector_type(4)));
typedef int dv4i_u __attribute__((ext_vector_type(4), aligned(8)));
typedef int dv2i __attribute__((ext_vector_type(2)));

// A slot's words (two pairs); two output pairs, one pair.
template <int PAST> __device__ __forceinline__ dv4i load_words(const dv4i *p)
{
    if constexpr (PAST == 2) return __builtin_nontemporal_load(p);
    else return *p;
}
template <int PAST> __device__ __forceinline__ void store_words(dv4i *p, dv4i v)
{
    if constexpr (PAST == 2) __builtin_nontemporal_store(v, p);
    else *p = v;
}
template <int PAST> __device__ __forceinline__ void store_two(int32_t *o, dv4i_u v)
{
    if constexpr (PAST > 0) __builtin_nontemporal_store(v, reinterpret_cast<dv4i_u *>(o));
    else *reinterpret_cast<dv4i_u *>(o) = v;
}
template <int PAST> __device__ __forceinline__ void store_one(int32_t *o, dv2i v)
{
    if constexpr (PAST > 0) __builtin_nontemporal_store(v, reinterpret_cast<dv2i *>(o));
    else *reinterpret_cast<dv2i *>(o) = v;
}

// Part `part` of tile (ti, tj) of one export.
template <bool CORR, int PAST>
__device__ __forceinline__ void dump_part(const DumpDesc &jd, int ti, int tj, int part, const PendingCorr &pc)
{
    constexpr int ROWS = DUMP_ROWS<PAST>;
    const int c = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = jd.n, nt = jd.nt;
    const int i0 = TILE * ti + ROWS * part;   // first row of the part
    if (ti == tj && part == 0) {
        // once per 128 inputs: the biases as of this reset, and the pre-sum
        // buffer the slot's next calls use
        const int j = TILE * ti + (int)threadIdx.x;
        if (jd.reset && threadIdx.x < TILE && j < n) base_of(jd, ti, 1 - jd.cur)[threadIdx.x] = jd.bias[j];
        if constexpr (CORR) {
            if (threadIdx.x < TILE && j < pc.n4) {
                pc.other[j] = 0;
                pc.other[pc.n4 + j] = 0;
            }
        }
        if (ti == 0 && threadIdx.x == 0 && jd.reset && jd.count != nullptr) *jd.count = 0;
    }
    const int cb = c >> 4, cj0 = 2 * (c & 15);
    const int j0 = TILE * tj + BLK * cb + cj0;
    const int ca = (ROWS * part) >> 5;        // block row
    // column block below the diagonal, or past the last input
    if (i0 >= n || j0 >= n || (ti == tj && cb < ca)) return;
    const int64_t tile = (int64_t)ti * nt - (int64_t)ti * (ti - 1) / 2 + (tj - ti);
    uint64_t *blk = reinterpret_cast<uint64_t *>(jd.acc) + tile * TILE_W + (ca * BLKS + cb) * BLOCK_W + cj0;
    constexpr int PER = ROWS / DUMP_WAVES;    // rows per wave
    dv4i w[PER];
    dv4i *pw[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int ra = (ROWS * part + wave + DUMP_WAVES * k) & (BLK - 1);   // row in the block
        pw[k] = reinterpret_cast<dv4i *>(blk + (4 * (ra >> 3) + (ra & 3)) * 64 + 32 * ((ra >> 2) & 1));
        w[k] = load_words<PAST>(pw[k]);
    }
    // the second column may lie past the last input: its bias is then that
    // of the first, and its pair is not stored
    const bool two = j0 + 1 < n;
    const int j1 = two ? j0 + 1 : j0;
    const int32_t *base = base_of(jd, tj, jd.cur);
    const uint32_t d0 = (uint32_t)jd.bias[j0] - (uint32_t)base[j0 - TILE * tj];
    const uint32_t d1 = (uint32_t)jd.bias[j1] - (uint32_t)base[j1 - TILE * tj];
    int64_t rj0 = 0, ij0 = 0, rj1 = 0, ij1 = 0;
    if constexpr (CORR) {
        rj0 = pc.sums[j0];
        ij0 = pc.sums[pc.n4 + j0];
        rj1 = pc.sums[j1];
        ij1 = pc.sums[pc.n4 + j1];
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int i = i0 + wave + DUMP_WAVES * k;
        if (i >= n) continue;
        if (jd.reset) store_words<PAST>(pw[k], dv4i{0, 0, 0, 0});
        uint64_t w0 = (uint64_t)(uint32_t)w[k].x | ((uint64_t)(uint32_t)w[k].y << 32);
        uint64_t w1 = (uint64_t)(uint32_t)w[k].z | ((uint64_t)(uint32_t)w[k].w << 32);
        if constexpr (CORR) {
            const int64_t ri = pc.sums[i], ii = pc.sums[pc.n4 + i];
            w0 += corr_word(ri, ii, rj0, ij0, pc.t);
            w1 += corr_word(ri, ii, rj1, ij1, pc.t);
        }
        const int a_re = pair_re(w0), a_im = (int32_t)((uint32_t)pair_im(w0) - d0);
        const int b_re = pair_re(w1), b_im = (int32_t)((uint32_t)pair_im(w1) - d1);
        int32_t *o = jd.out + 2 * ((int64_t)i * n - (int64_t)i * (i - 1) / 2 + (j0 - i));
        if (j0 >= i && two)
            store_two<PAST>(o, dv4i_u{a_re, a_im, b_re, b_im});
        else if (j0 >= i)
            store_one<PAST>(o, dv2i{a_re, a_im});
        else if (j0 + 1 >= i && two)
            store_one<PAST>(o + 2, dv2i{b_re, b_im});
    }
}

// One slot's export: workgroup x is part x % DUMP_PARTS of tile
// x / DUMP_PARTS of the triangle.
template <bool CORR, int PAST>
__global__ __launch_bounds__(64 * DUMP_WAVES) void vis_dump(DumpDesc jd, PendingCorr pc)
{
    int ti, tj;
    tile_of((int)(blockIdx.x / DUMP_PARTS<PAST>), jd.nt, ti, tj);
    dump_part<CORR, PAST>(jd, ti, tj, (int)(blockIdx.x % DUMP_PARTS<PAST>), pc);
}

// Batched export: the jobs' tiles one after another, tile g being tile
// g - first_tile of its job.  The job of a tile comes from the table
// `job_of` (one entry per tile), or, with no table, every job having
// `tiles` of them, by division.
template <int PAST>
__global__ __launch_bounds__(64 * DUMP_WAVES) void vis_dump_batch(const DumpDesc *__restrict__ jobs,
                                                                  const int32_t *__restrict__ job_of, int tiles)
{
    const int g = (int)(blockIdx.x / DUMP_PARTS<PAST>);
    const int k = __builtin_amdgcn_readfirstlane(job_of ? job_of[g] : g / tiles);
    const DumpDesc jd = jobs[k];
    int ti, tj;
    tile_of(g - jd.first_tile, jd.nt, ti, tj);
    dump_part<false, PAST>(jd, ti, tj, (int)(blockIdx.x % DUMP_PARTS<PAST>), PendingCorr{nullptr, nullptr, 0, 0});
}

// Ingest of host-sourced frames (the streaming server): up to GATHER_MAX
// frames of `words` 16-byte words each, every frame from pinned host memory
// (read over PCIe by the workgroups themselves, no DMA-engine copy) into
// device memory.  Workgroups (x, f) share frame f; each thread keeps eight
// 16-byte loads in flight.
constexpr int GATHER_MAX = 120;
constexpr int GATHER_WGS_PER_FRAME = 4;
typedef unsigned int gv4u __attribute__((ext_vector_type(4)));
struct GatherArgs {
    int32_t n;                       // frames
    int32_t words;                   // 16-byte words per frame
    const gv4u *src[GATHER_MAX];     // device-visible addresses of pinned host frames
    gv4u *dst[GATHER_MAX];
};

__global__ __launch_bounds__(256) void gather_frames(GatherArgs a)
{
    const gv4u *__restrict__ src = a.src[blockIdx.y];
    gv4u *__restrict__ dst = a.dst[blockIdx.y];
    const int step = (int)(blockDim.x * gridDim.x);
    int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    for (; i + 7 * step < a.words; i += 8 * step) {
        gv4u v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = src[i + k * step];
#pragma unroll
        for (int k = 0; k < 8; ++k) dst[i + k * step] = v[k];
    }
    for (; i < a.words; i += step) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void fill_zero(int4 *__restrict__ p, int64_t n4)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < n4;
         k += (int64_t)gridDim.x * 256)
        p[k] = make_int4(0, 0, 0, 0);
}

// A slot cleared without an export: its accumulators (with the bases of its
// biases), its biases (n_bias int32, a multiple of 4), and, if given, its
// device sample counter.
__global__ __launch_bounds__(256) void clear_slot(int4 *__restrict__ acc, int64_t n4, int4 *__restrict__ bias,
                                                  int n_bias4, int64_t *count)
{
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int64_t k = first; k < n4; k += step) acc[k] = make_int4(0, 0, 0, 0);
    for (int64_t k = first; k < n_bias4; k += step) bias[k] = make_int4(0, 0, 0, 0);
    if (first == 0 && count != nullptr) *count = 0;
}

// Integration guard of a prepared batch, run ahead of its correlation
// launches: if every job's slot can take its samples without passing T_MAX,
// the counters advance and *skip = 0; otherwise nothing changes, *skip = 1
// (the correlation launches then return at once) and *skipped counts the
// refusal.  One workgroup: every thread checks its share of the jobs, the
// verdict is agreed at a barrier before any counter moves, and the jobs'
// counters are distinct (a batch names each slot once), so each thread
// advances its own.
__global__ __launch_bounds__(1024) void batch_guard(const GuardJob *__restrict__ jobs, int n_jobs, int32_t *skip,
                                                    int64_t *skipped)
{
    bool ok = true;
    for (int k = threadIdx.x; k < n_jobs; k += blockDim.x) ok = ok && jobs[k].n <= T_MAX - *jobs[k].count;
    ok = __syncthreads_and(ok ? 1 : 0) != 0;
    if (ok)
        for (int k = threadIdx.x; k < n_jobs; k += blockDim.x) *jobs[k].count += jobs[k].n;
    if (threadIdx.x == 0) {
        if (!ok) *skipped += 1;
        *skip = ok ? 0 : 1;
    }
}

// Stores one value into a device sample counter, in stream order.
__global__ void set_count(int64_t *p, int64_t v)
{
    if (threadIdx.x == 0) *p = v;
}

// Scalar reference: one thread per pair (i <= j), int32 sums over t.
__global__ __launch_bounds__(256) void xcorr_scalar(const uint8_t *__restrict__ s, int64_t n_samples,
                                                    int n, int64_t stride, uint32_t re_low,
                                                    int32_t *__restrict__ out)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t npairs = (int64_t)n * (n + 1) / 2;
    if (k >= npairs) return;
    const double b = 2.0 * n + 1.0;
    int i = (int)floor((b - sqrt(b * b - 8.0 * (double)k)) * 0.5);
    auto row_start = [n](int64_t r) { return r * n - r * (r - 1) / 2; };
    if (i < 0) i = 0;
    if (i > n - 1) i = n - 1;
    while (i + 1 < n && row_start(i + 1) <= k) ++i;
    while (i > 0 && row_start(i) > k) --i;
    const int j = i + (int)(k - row_start(i));
    int32_t vr = 0, vi = 0;
    for (int64_t t = 0; t < n_samples; ++t) {
        const uint32_t bi = s[t * stride + i], bj = s[t * stride + j];
        const int hi_i = (int)(bi >> 4) - 8, lo_i = (int)(bi & 15u) - 8;
        const int hi_j = (int)(bj >> 4) - 8, lo_j = (int)(bj & 15u) - 8;
        const int ri = re_low ? lo_i : hi_i, ii = re_low ? hi_i : lo_i;
        const int rj = re_low ? lo_j : hi_j, ij = re_low ? hi_j : lo_j;
        vr += ri * rj + ii * ij;
        vi += ii * rj - ri * ij;
    }
    out[2 * k] = vr;
    out[2 * k + 1] = vi;
}

// ---------------------------------------------------------------------------
// Launchers (host)
// ---------------------------------------------------------------------------
// `aligned`: every job's samples pointer and row stride are multiples of 4
// bytes and its N is a multiple of 4, so whole dwords can be loaded.
hipError_t launch_correlate(const KernelArgs &a, int grid, bool aligned, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    if (aligned)
        hipLaunchKernelGGL((xcorr_mfma<true, false, false>), dim3(grid), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((xcorr_mfma<false, false, false>), dim3(grid), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// The exact FP8 path: the same kernel with E4M3 operands and fp32 sums
// (pieces below 2^17 samples).
hipError_t launch_correlate_fp8(const KernelArgs &a, int grid, bool aligned, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    if (aligned)
        hipLaunchKernelGGL((xcorr_mfma<true, false, true>), dim3(grid), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((xcorr_mfma<false, false, true>), dim3(grid), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// The unsigned-nibble form (xeng_correlate_presum): the same kernel on the
// stored nibbles; its sums need the pre-sum correction below.
hipError_t launch_correlate_unsigned(const KernelArgs &a, int grid, bool aligned, hipStream_t stream)
{
    if (grid <= 0) return hipSuccess;
    if (aligned)
        hipLaunchKernelGGL((xcorr_mfma<true, true, false>), dim3(grid), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL((xcorr_mfma<false, true, false>), dim3(grid), dim3(256), 0, stream, a);
    return hipGetLastError();
}

// The form (PAST) of a launch whose resetting exports hold this many tiles:
// go(std::integral_constant<int, PAST>).
template <typename Go> static hipError_t with_dump_form(int64_t reset_tiles, Go go)
{
    const int64_t bytes = reset_tiles * TILE_I32 * (int64_t)sizeof(int32_t);
    if (bytes >= DUMP_PAST_BYTES) go(std::integral_constant<int, 2>());
    else if (bytes >= STREAM_BYTES) go(std::integral_constant<int, 1>());
    else go(std::integral_constant<int, 0>());
    return hipGetLastError();
}

hipError_t launch_dump(const DumpDesc &jd, hipStream_t stream)
{
    const int64_t tiles = (int64_t)jd.nt * (jd.nt + 1) / 2;
    return with_dump_form(jd.reset ? tiles : 0, [&](auto form) {
        constexpr int PAST = decltype(form)::value;
        hipLaunchKernelGGL((vis_dump<false, PAST>), dim3((unsigned)(tiles * DUMP_PARTS<PAST>)), dim3(64 * DUMP_WAVES), 0,
                           stream, jd, PendingCorr{nullptr, nullptr, 0, 0});
    });
}

// A resetting export that also applies a slot's pending unsigned-form
// correction (`sums`: its SR, SI over `t` samples, n4 apart) and clears
// `other`.
hipError_t launch_dump_corr(const DumpDesc &jd, const int32_t *sums, int n4, int64_t t, int32_t *other,
                            hipStream_t stream)
{
    const int64_t tiles = (int64_t)jd.nt * (jd.nt + 1) / 2;
    return with_dump_form(tiles, [&](auto form) {
        constexpr int PAST = decltype(form)::value;
        hipLaunchKernelGGL((vis_dump<true, PAST>), dim3((unsigned)(tiles * DUMP_PARTS<PAST>)), dim3(64 * DUMP_WAVES), 0,
                           stream, jd, PendingCorr{sums, other, n4, t});
    });
}

// `d_jobs`: descriptors in device memory, `total_tiles` tiles in all (at most
// DUMP_MAX_TILES), `reset_tiles` of them of resetting exports; d_job_of: the
// job of each tile, or null where every job has `tiles`.
hipError_t launch_dump_batch(const DumpDesc *d_jobs, const int32_t *d_job_of, int tiles, int64_t total_tiles,
                             int64_t reset_tiles, hipStream_t stream)
{
    static_assert(DUMP_MAX_TILES * DUMP_PARTS<2> < (INT64_C(1) << 31), "a launch's workgroups fit its grid");
    if (total_tiles <= 0) return hipSuccess;
    return with_dump_form(reset_tiles, [&](auto form) {
        constexpr int PAST = decltype(form)::value;
        hipLaunchKernelGGL(vis_dump_batch<PAST>, dim3((unsigned)(total_tiles * DUMP_PARTS<PAST>)), dim3(64 * DUMP_WAVES),
                           0, stream, d_jobs, d_job_of, tiles);
    });
}

// `n` frames of `bytes` each (a multiple of 16, below 2^31), every address
// 16-byte aligned; any number of frames (GATHER_MAX per launch).
hipError_t launch_gather_frames(const uint8_t *const *src, uint8_t *const *dst, int n, int64_t bytes,
                                hipStream_t stream)
{
    for (int f0 = 0; f0 < n; f0 += GATHER_MAX) {
        GatherArgs a;
        a.n = std::min(GATHER_MAX, n - f0);
        a.words = (int32_t)(bytes / 16);
        for (int k = 0; k < a.n; ++k) {
            a.src[k] = reinterpret_cast<const gv4u *>(src[f0 + k]);
            a.dst[k] = reinterpret_cast<gv4u *>(dst[f0 + k]);
        }
        hipLaunchKernelGGL(gather_frames, dim3(GATHER_WGS_PER_FRAME, (unsigned)a.n), dim3(256), 0, stream, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_zero(int32_t *p, int64_t n_i32, hipStream_t stream)
{
    const int64_t n4 = n_i32 / 4;
    if (n4 <= 0) return hipSuccess;
    int64_t blocks = (n4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_zero, dim3((unsigned)blocks), dim3(256), 0, stream,
                       reinterpret_cast<int4 *>(p), n4);
    return hipGetLastError();
}

hipError_t launch_clear_slot(int32_t *acc, int64_t n_i32, int32_t *bias, int64_t n_bias, int64_t *count,
                             hipStream_t stream)
{
    const int64_t n4 = n_i32 / 4;
    int64_t blocks = (n4 + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(clear_slot, dim3((unsigned)blocks), dim3(256), 0, stream, reinterpret_cast<int4 *>(acc), n4,
                       reinterpret_cast<int4 *>(bias), (int)(n_bias / 4), count);
    return hipGetLastError();
}

hipError_t launch_batch_guard(const GuardJob *d_jobs, int n_jobs, int32_t *d_skip, int64_t *d_skipped,
                              hipStream_t stream)
{
    const int threads = std::min(1024, std::max(64, (n_jobs + 63) / 64 * 64));
    hipLaunchKernelGGL(batch_guard, dim3(1), dim3(threads), 0, stream, d_jobs, n_jobs, d_skip, d_skipped);
    return hipGetLastError();
}

hipError_t launch_set_count(int64_t *p, int64_t v, hipStream_t stream)
{
    hipLaunchKernelGGL(set_count, dim3(1), dim3(64), 0, stream, p, v);
    return hipGetLastError();
}

hipError_t launch_reference(const uint8_t *s, int64_t n_samples, int n, int64_t stride,
                            uint32_t re_low, int32_t *out, hipStream_t stream)
{
    const int64_t npairs = (int64_t)n * (n + 1) / 2;
    const int64_t blocks = (npairs + 255) / 256;
    hipLaunchKernelGGL(xcorr_scalar, dim3((unsigned)blocks), dim3(256), 0, stream, s, n_samples,
                       n, stride, re_low, out);
    return hipGetLastError();
}

}  // namespace xeng
