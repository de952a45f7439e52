// Flag-aware correlation and its RFI-excision step (the "RFI Excision" task
// of Table tab:computing; the flags and metadata that travel with every
// block of samples, Sec. 2.2).
//
// A flag covers one input over a block of L consecutive samples of a call.
// Flagged samples enter no visibility (they are replaced by the zero sample
// while the call's samples are copied into padded rows for the wide
// correlation kernel), and every pair counts the samples at which neither
// of its inputs was flagged:
//     n_ij = sum_b len_b * w_i(b) * w_j(b),   w = 1 - flag,
// kept per slot in int32 (n_ij <= T_MAX).  The counts come from bit-packed
// "unflagged" masks, 32 blocks per word: n_ij = L * popcount(w_i & w_j)
// over the full blocks, plus the last block's length if both are unflagged
// there.
//
// RFI excision: the spectral kurtosis of the M samples of each (block,
// input), from the power P = |x|^2 (Nita & Gary 2010),
//     SK = (M + 1) / (M - 1) * (M S2 / S1^2 - 1),  S1 = sum P, S2 = sum P^2,
// flagged when below lo or above hi (integer fractions over one
// denominator), or when S1 = 0.  The comparison is exact in 64-bit
// integers: with M <= 1024 and |P| <= 128, M S2 <= 2^34 and S1^2 <= 2^34, so
// both sides stay below 2^58 for thresholds up to 16.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "xeng_internal.h"
#include "xeng_rows.h"

namespace xeng {

// Power sums of one byte (one complex sample) into s1, s2.
__device__ __forceinline__ void power_sums(uint32_t byte, int sh_re, int sh_im, int32_t &s1, int32_t &s2)
{
    const int re = (int)((byte >> sh_re) & 15u) - 8, im = (int)((byte >> sh_im) & 15u) - 8;
    const int p = re * re + im * im;
    s1 += p;
    s2 += p * p;
}

// The flag decision of one (block, input) from its sums over m samples.
__device__ __forceinline__ uint8_t sk_decide(int32_t s1, int32_t s2, int m, int64_t lo_num, int64_t hi_num,
                                             int64_t den)
{
    if (m < 2) return 0;
    if (s1 == 0) return 1;
    const int64_t a = s1, q = (int64_t)m * s2 - a * a;
    const int64_t num = (int64_t)(m + 1) * q, dd = (int64_t)(m - 1) * a * a;
    return (num * den < lo_num * dd || num * den > hi_num * dd) ? 1 : 0;
}

// Squares of the offset-decoded nibbles u - 8 of four bytes each holding one
// nibble's low three bits in `idx` (0..7) and, in `top`, 0xFF where its bit 3
// is set: (idx)^2 there, else (idx - 8)^2, by byte permutes of two 8-entry
// tables.
__device__ __forceinline__ uint32_t nib_squares(uint32_t idx, uint32_t top)
{
    const uint32_t pos = __builtin_amdgcn_perm(0x31241910u, 0x09040100u, idx);   // 0 1 4 9 16 25 36 49
    const uint32_t neg = __builtin_amdgcn_perm(0x01040910u, 0x19243140u, idx);   // 64 49 36 25 16 9 4 1
    return (pos & top) | (neg & ~top);
}

// Four samples of one input (a byte each): their powers' sums into s1, s2.
// A byte permute with selectors 8..11 replicates the sign bits of bytes 1, 3,
// 5 and 7 of its two sources; with the word and the word shifted up a byte
// those are the four bytes' top bits.
__device__ __forceinline__ void power_sums4(uint32_t x, uint32_t &s1, uint32_t &s2)
{
    constexpr uint32_t TOP = 0x0B090A08u;
    const uint32_t hi = nib_squares((x >> 4) & 0x07070707u, __builtin_amdgcn_perm(x, x << 8, TOP));
    const uint32_t lo = nib_squares(x & 0x07070707u, __builtin_amdgcn_perm(x << 4, x << 12, TOP));
    const uint32_t p = hi + lo;   // at most 128 in a byte
    s1 = __builtin_amdgcn_udot4(p, 0x01010101u, s1, false);
    s2 = __builtin_amdgcn_udot4(p, p, s2, false);
}

// A workgroup takes 16 CW inputs x one block of rows, any alignment and N >=
// 16: a lane holds a chunk of 16 inputs (the row's last 16 for a chunk that
// would pass its end: those inputs' sums are then formed twice, alike) and
// takes four rows at a time, one 16-byte load each, transposed by byte
// permutes so that a register holds four samples of one input.  The 64 / CW
// row groups of every wave take the block's row quads in turn; their sums
// meet in LDS by atomic adds, and one thread per input takes the exact
// decision.
//
// Bound by HBM: every sample byte is read once, at 4.8 integer operations a
// sample (one sample per operation and input before: some ten).  N = 2048, T =
// 32768, 256-sample blocks (67 MB): 27.3 -> 18.3 us = 3.7 TB/s (eight waves a
// workgroup 18.3, four 21.1, two 32.6: one workgroup per CU there, whose first
// loads and last sums nothing overlaps); N = 500 (unaligned rows, byte loads
// before), T = 8192: 41 -> 8.8 us.
template <int CW>
__global__ __launch_bounds__(1024) void sk_flags_vec(const uint8_t *__restrict__ s, int64_t n_samples, int n,
                                                     int64_t stride, int block_len, int64_t lo_num, int64_t hi_num,
                                                     int64_t den, uint8_t *__restrict__ flags)
{
    constexpr int GROUPS = 64 / CW;
    __shared__ uint32_t sum[32 * CW];   // [S1, S2][input of a chunk][chunk]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int c = lane % CW, c0 = CW * (int)blockIdx.x;
    const int64_t b = blockIdx.y;
    const int64_t t0 = b * block_len;
    const int m = (int)(t0 + block_len < n_samples ? block_len : n_samples - t0);
    for (int k = threadIdx.x; k < 32 * CW; k += blockDim.x) sum[k] = 0;
    __syncthreads();
    if (16 * (c0 + c) < n) {
        const uint8_t *p = s + t0 * stride + min(16 * (c0 + c), n - 16);
        uint32_t s1[16], s2[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) s1[k] = s2[k] = 0;
        const int quads = (m + 3) / 4, step = waves * GROUPS;
        auto load = [&](row16 (&v)[4], int q) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // rows past the block's end: the zero sample, no power
                v[u] = row16{0x88888888u, 0x88888888u, 0x88888888u, 0x88888888u};
                if (4 * q + u < m) v[u] = *reinterpret_cast<const row16_u *>(p + (int64_t)(4 * q + u) * stride);
            }
        };
        auto use = [&](const row16 (&v)[4]) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t ab_lo = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x05010400u);
                const uint32_t ab_hi = __builtin_amdgcn_perm(v[1][w], v[0][w], 0x07030602u);
                const uint32_t cd_lo = __builtin_amdgcn_perm(v[3][w], v[2][w], 0x05010400u);
                const uint32_t cd_hi = __builtin_amdgcn_perm(v[3][w], v[2][w], 0x07030602u);
                power_sums4(__builtin_amdgcn_perm(cd_lo, ab_lo, 0x05040100u), s1[4 * w], s2[4 * w]);
                power_sums4(__builtin_amdgcn_perm(cd_lo, ab_lo, 0x07060302u), s1[4 * w + 1], s2[4 * w + 1]);
                power_sums4(__builtin_amdgcn_perm(cd_hi, ab_hi, 0x05040100u), s1[4 * w + 2], s2[4 * w + 2]);
                power_sums4(__builtin_amdgcn_perm(cd_hi, ab_hi, 0x07060302u), s1[4 * w + 3], s2[4 * w + 3]);
            }
        };
        row16 v0[4], v1[4];
        int q = wave * GROUPS + lane / CW;
        load(v0, q);
        for (; q < quads; q += 2 * step) {
            load(v1, q + step);
            use(v0);
            load(v0, q + 2 * step);
            use(v1);
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            atomicAdd(&sum[k * CW + c], s1[k]);
            atomicAdd(&sum[(16 + k) * CW + c], s2[k]);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 16 * CW; e += blockDim.x) {
        const int ch = e / 16, k = e % 16, first = 16 * (c0 + ch);
        if (first >= n) continue;
        flags[b * n + min(first, n - 16) + k] =
            sk_decide((int32_t)sum[k * CW + ch], (int32_t)sum[(16 + k) * CW + ch], m, lo_num, hi_num, den);
    }
}

// One thread per (input, block), byte loads.
__global__ __launch_bounds__(256) void sk_flags_bytes(const uint8_t *__restrict__ s, int64_t n_samples, int n,
                                                      int64_t stride, uint32_t re_low, int block_len, int64_t lo_num,
                                                      int64_t hi_num, int64_t den, uint8_t *__restrict__ flags)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    const int64_t b = blockIdx.y;
    if (i >= n) return;
    const int64_t t0 = b * block_len;
    const int64_t t1 = t0 + block_len < n_samples ? t0 + block_len : n_samples;
    const int sh_re = re_low ? 0 : 4, sh_im = re_low ? 4 : 0;
    int32_t s1 = 0, s2 = 0;
    for (int64_t t = t0; t < t1; ++t) power_sums(s[t * stride + i], sh_re, sh_im, s1, s2);
    flags[b * n + i] = sk_decide(s1, s2, (int)(t1 - t0), lo_num, hi_num, den);
}

// Rows of n samples (any stride and alignment) copied into rows `pitch` bytes
// apart, each n16 = n rounded up to 16 bytes padded with the zero sample: a
// layout the DMA kernels read.  MASK: every sample of a flagged (block, input)
// becomes the zero sample; row t of the copy is sample t_first + t of the
// call, in block (t_first + t) / block_len.
//
// Bound by HBM: 2 N bytes a row.  A workgroup takes consecutive rows, 2^xs
// threads side by side on a row, a thread 16 bytes of R rows (all loads before
// the first store).  Several rows a thread where that leaves COPY_WGS
// workgroups, eight per compute unit: N = 1000, T = 32768 16.0 us (a dword per
// thread, a row per workgroup) -> 12.5 us with four rows (13.1 with two, 13.8
// with one); with flags, N = 2048, T = 32768 (134 MB) 21.0 us with two (22.0
// with one, 22.3 with four, 20.6 for the aligned-only form it replaces), N =
// 500, T = 8192 10.1 -> 9.7 us.  One row a thread below that, where few
// workgroups wait on one row after the other: a batch of 16 jobs of N = 1000,
// T = 256 131 us (four rows 155), T = 8192 313 (336); N = 300, T = 16384 141
// (159).
__device__ __forceinline__ uint32_t mask_word(uint32_t x, uint32_t f)
{
    // bytes of f that are nonzero -> 0xFF
    const uint32_t hi = ((f & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | f;
    const uint32_t m = ((hi >> 7) & 0x01010101u) * 0xFFu;
    return (x & ~m) | (0x88888888u & m);
}

constexpr int COPY_WGS = 2048;

template <bool MASK, int R>
__global__ __launch_bounds__(256) void copy_rows(const uint8_t *__restrict__ src, int64_t stride, int n, int64_t rows,
                                                 uint8_t *__restrict__ dst, int64_t pitch, int xs,
                                                 const uint8_t *__restrict__ flags, int block_len, int64_t t_first)
{
    const int x = threadIdx.x & ((1 << xs) - 1), y = threadIdx.x >> xs, ny = 256 >> xs;
    for (int64_t t0 = (int64_t)blockIdx.x * ny * R + y; t0 < rows; t0 += (int64_t)gridDim.x * ny * R)
        for (int c = 16 * x; c < n; c += 16 << xs) {
            row16 v[R], f[R];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int64_t t = t0 + k * ny;
                if (t >= rows) continue;
                v[k] = load_row16(src + t * stride, c, n);
                if (MASK) {
                    const uint32_t b = (uint32_t)(t_first + t) / (uint32_t)block_len;   // T_MAX samples at most
                    f[k] = load_row16(flags + (int64_t)b * n, c, n);
                }
            }
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const int64_t t = t0 + k * ny;
                if (t >= rows) continue;
                if (MASK)
#pragma unroll
                    for (int w = 0; w < 4; ++w) v[k][w] = mask_word(v[k][w], f[k][w]);
                *reinterpret_cast<row16 *>(dst + t * pitch + c) = v[k];
            }
        }
}

// Unflagged masks packed along blocks: bits[i][w] bit k set when block
// 32 w + k of input i is unflagged.  One wave per (two inputs, word): lane l
// reads block 32 w + l % 32 of input i0 + l / 32, and one ballot of the
// unflagged lanes holds both inputs' words.
__global__ __launch_bounds__(256) void pack_unflagged(const uint8_t *__restrict__ flags, int nb, int n, int words,
                                                      uint32_t *__restrict__ bits)
{
    const int lane = (int)threadIdx.x & 63;
    const int64_t wv = (int64_t)blockIdx.x * 4 + ((int)threadIdx.x >> 6);
    const int64_t pairs = (n + 1) / 2;
    if (wv >= pairs * words) return;   // whole waves
    const int w = (int)(wv % words), i0 = 2 * (int)(wv / words);
    const int i = i0 + (lane >> 5), b = 32 * w + (lane & 31);
    const bool unflagged = i < n && b < nb && flags[(int64_t)b * n + i] == 0;
    const uint64_t m = __ballot(unflagged);
    if (lane == 0) bits[(int64_t)i0 * words + w] = (uint32_t)m;
    if (lane == 32 && i < n) bits[(int64_t)i * words + w] = (uint32_t)(m >> 32);
}

// Per-pair sample counts added into counts[k(i, j)] (packed upper triangle).
// A workgroup takes a 64 x 64 block of pairs (row block by, column block
// bx >= by); thread (ty, tx) takes rows 4 ty .. + 3 and columns tx + 16 q
// (q < 4), so that each row's 64 counts are updated by 16 consecutive
// threads at a time.  The masks of the 64 + 64 inputs go through LDS in
// chunks of up to CW words.  Blocks 0 .. nb-2 weigh block_len each, the
// last `last_len`.  `fresh`: the counts hold nothing since the slot's reset
// (which leaves them as they are) and are stored, not read.
constexpr int CW = 32;
__global__ __launch_bounds__(256) void count_pairs(const uint32_t *__restrict__ bits, int words, int nb, int n,
                                                   int block_len, int last_len, int fresh,
                                                   int32_t *__restrict__ counts)
{
    const int by = blockIdx.y, bx = blockIdx.x;
    if (bx < by) return;
    __shared__ uint32_t ra[64][CW + 1], cb[64][CW + 1];
    const int tid = threadIdx.x;
    const int ty = tid >> 4, tx = tid & 15;
    int32_t c[4][4] = {};
    const int last_w = (nb - 1) >> 5;
    const uint32_t last_bit = 1u << ((nb - 1) & 31);
    for (int w0 = 0; w0 < words; w0 += CW) {
        const int cw = words - w0 < CW ? words - w0 : CW;
        for (int e = tid; e < 64 * cw; e += 256) {
            const int r = e / cw, w = e % cw;
            const int ia = 64 * by + r, ib = 64 * bx + r;
            ra[r][w] = ia < n ? bits[(int64_t)ia * words + w0 + w] : 0u;
            cb[r][w] = ib < n ? bits[(int64_t)ib * words + w0 + w] : 0u;
        }
        __syncthreads();
        for (int w = 0; w < cw; ++w) {
            // the last block counts with its own length, below
            const uint32_t keep = (w0 + w == last_w) ? ~last_bit : 0xFFFFFFFFu;
            uint32_t a[4], b[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                a[k] = ra[4 * ty + k][w] & keep;
                b[k] = cb[tx + 16 * k][w];
            }
#pragma unroll
            for (int p = 0; p < 4; ++p)
#pragma unroll
                for (int q = 0; q < 4; ++q) c[p][q] += __popc(a[p] & b[q]);
        }
        __syncthreads();
    }
    bool lj[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int j = 64 * bx + tx + 16 * q;
        lj[q] = j < n && (bits[(int64_t)j * words + last_w] & last_bit) != 0;
    }
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int i = 64 * by + 4 * ty + p;
        if (i >= n) continue;
        const bool li = (bits[(int64_t)i * words + last_w] & last_bit) != 0;
        const int64_t row = (int64_t)i * n - (int64_t)i * (i - 1) / 2 - i;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int j = 64 * bx + tx + 16 * q;
            if (j >= n || j < i) continue;
            const int32_t v = c[p][q] * block_len + ((li && lj[q]) ? last_len : 0);
            counts[row + j] = fresh ? v : counts[row + j] + v;
        }
    }
}

// out[k] = counts[k] + base (samples integrated without flags count for
// every pair); `counts` null: no flagged samples since the slot's reset.
__global__ __launch_bounds__(256) void counts_export(const int32_t *__restrict__ counts, int64_t npairs, int32_t base,
                                                     int32_t *__restrict__ out)
{
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < npairs; k += (int64_t)gridDim.x * 256)
        out[k] = (counts ? counts[k] : 0) + base;
}

hipError_t launch_sk_flags(const uint8_t *s, int64_t n_samples, int n, int64_t stride, uint32_t re_low,
                           int block_len, int64_t lo_num, int64_t hi_num, int64_t den, uint8_t *flags,
                           hipStream_t stream)
{
    const int64_t nb = (n_samples + block_len - 1) / block_len;
    if (nb <= 0) return hipSuccess;
    // The byte form for N < 16 and for blocks too small for a workgroup of
    // the other: its LDS sums and barriers then cost more than the block's
    // samples.  Byte form / other, us: N = 1000, T = 16384, blocks of two 22 /
    // 29; T = 32768, N = 64, of 4 6.6 / 20, of 16 6.6 / 7.5; N = 500, of 4 16 /
    // 20, of 8 14.0 / 12.3; N = 1000, of 4 33 / 29; and for blocks up to eight
    // while the samples are few: N = 1000, T = 8192, of 3 8.3 / 13.4, of 8 6.5 /
    // 8.9, of 16 6.5 / 7.6; N = 2048, T = 8192, of 8 9.5 / 10.9, T = 32768 52 / 30.
    if (n < 16 || block_len <= 2 || (block_len <= 16 && n * block_len < 3000) ||
        (block_len <= 8 && n * n_samples <= 1 << 24)) {
        hipLaunchKernelGGL(sk_flags_bytes, dim3((unsigned)((n + 255) / 256), (unsigned)nb), dim3(256), 0, stream, s,
                           n_samples, n, stride, re_low, block_len, lo_num, hi_num, den, flags);
        return hipGetLastError();
    }
    // the narrowest row of lanes that holds the inputs' chunks, and a wave
    // for every two row quads of each of its row groups, up to 16
    const int chunks = (n + 15) / 16;
    auto go = [&](auto kernel, int cw) {
        const int per_wave = 4 * 2 * (64 / cw);
        const int waves = std::min(16, std::max(1, (block_len + per_wave - 1) / per_wave));
        hipLaunchKernelGGL(kernel, dim3((unsigned)((chunks + cw - 1) / cw), (unsigned)nb), dim3(64 * waves), 0, stream,
                           s, n_samples, n, stride, block_len, lo_num, hi_num, den, flags);
    };
    if (chunks <= 4) go(sk_flags_vec<4>, 4);
    else if (chunks <= 16) go(sk_flags_vec<16>, 16);
    else if (chunks <= 32) go(sk_flags_vec<32>, 32);
    else go(sk_flags_vec<64>, 64);
    return hipGetLastError();
}

// `dst`: rows `pitch` bytes apart (a multiple of 16, >= n), 16-byte aligned;
// `flags` null: a plain padded copy.
hipError_t launch_copy_rows(const uint8_t *src, int64_t stride, int n, int64_t rows, uint8_t *dst, int64_t pitch,
                            const uint8_t *flags, int block_len, int64_t t_first, hipStream_t stream)
{
    if (rows <= 0) return hipSuccess;
    const int per_row = (n + 15) / 16;
    int xs = 0;
    while (xs < 8 && (1 << xs) < per_row) ++xs;
    const int64_t one = (rows + (256 >> xs) - 1) / (256 >> xs);   // workgroups of one row a thread
    auto go = [&](auto kernel, int r) {
        const int64_t blocks = std::min<int64_t>(65535, (one + r - 1) / r);
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, src, stride, n, rows, dst, pitch, xs,
                           flags, block_len, t_first);
    };
    if (flags && one >= 2 * COPY_WGS) go(copy_rows<true, 2>, 2);
    else if (flags) go(copy_rows<true, 1>, 1);
    else if (one >= 4 * COPY_WGS) go(copy_rows<false, 4>, 4);
    else go(copy_rows<false, 1>, 1);
    return hipGetLastError();
}

hipError_t launch_counts(const uint8_t *flags, int nb, int n, int block_len, int last_len, uint32_t *bits,
                         int32_t *counts, bool fresh, hipStream_t stream)
{
    if (nb <= 0) return hipSuccess;
    const int words = (nb + 31) / 32;
    const int64_t waves = (int64_t)((n + 1) / 2) * words;   // one per (two inputs, word)
    hipLaunchKernelGGL(pack_unflagged, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, stream, flags, nb, n, words,
                       bits);
    const unsigned tiles = (unsigned)((n + 63) / 64);
    hipLaunchKernelGGL(count_pairs, dim3(tiles, tiles), dim3(256), 0, stream, bits, words, nb, n, block_len,
                       last_len, fresh ? 1 : 0, counts);
    return hipGetLastError();
}

hipError_t launch_counts_export(const int32_t *counts, int64_t npairs, int32_t base, int32_t *out,
                                hipStream_t stream)
{
    if (npairs <= 0) return hipSuccess;
    int64_t blocks = (npairs + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(counts_export, dim3((unsigned)blocks), dim3(256), 0, stream, counts, npairs, base, out);
    return hipGetLastError();
}

}  // namespace xeng
