// Phased-array beamforming (Sec. 2.1: the nodes form 10 phased-array beams
// for pulsar timing from the channelised samples; "Pulsar Beamforming" in
// Table tab:computing):
//     y_b(t) = sum_i w_bi x_i(t),
// complex int8 weights (parts in [-127, 127]) and 4+4-bit samples, exact
// int32 sums.  Per time sample this is a [1 x 2N] by [2N x 2B] real
// product, so a block of 16 time rows against up to 16 beams is one
// v_mfma_i32_16x16x64_i8 per 32 inputs and per output part:
//   A (rows = times)  : (Re x_i, -Im x_i) for Re y, (Im x_i, Re x_i) for Im y,
//                       8 inputs per lane and step, both formed in registers
//   B (cols = beams)  : (Re w, Im w) pairs, for both.
// The kernel reads every sample once, so it is bound by HBM bandwidth (about
// 10 complex MACs per sample byte for 10 beams), not by the matrix cores:
// N = 2048, T = 32768, 10 beams (69.7 MB) 13.8 us, the 5.1 TB/s that a large
// copy reaches.  What the time had gone on besides: 128 KiB
// of weights per workgroup (both parts' operands), loaded before the first
// sample, one workgroup per CU (17.6 us); and byte loads for rows that are
// not 16-byte aligned (N = 1000, T = 16384, 16 beams 7.2 us, was 45.6).
//
// Workgroup: 32 or 64 time rows, 16 per wave or pair of waves, persistent over
// row blocks; the
// weights of up to 2048 inputs sit in LDS in operand order (32 B per input:
// 16 beams x 2 parts), loaded once, or per chunk of 2048 inputs when N is
// larger; two or more workgroups share a CU.  The first samples are requested
// right behind the weights, and the barrier waits for the weights only.  A lane
// loads 16 bytes (16 inputs of its row, at any byte address) per pair of
// k-steps; the k index of a byte is (step, lane group, position), the same for
// A and B.
#include <hip/hip_runtime.h>

#include "xeng_internal.h"
#include "xeng_rows.h"

namespace xeng {

typedef int bv4i __attribute__((ext_vector_type(4)));

constexpr int BEAM_CHUNK = 2048;                  // inputs whose weights fit in LDS
constexpr int BEAM_IN_BYTES = 32;                 // LDS bytes per input: 16 beams x (re, im)
constexpr int BEAM_LDS = BEAM_CHUNK * BEAM_IN_BYTES;   // 64 KiB
constexpr int BEAMS_MAX = 16;
constexpr int BEAM_PAIR = 64;                     // inputs of a pair of k-steps

// The offset-decoded nibbles of 4 packed samples as int8 pairs, two dwords
// for each output part: (re, -im) and (im, re).
__device__ __forceinline__ void unpack4(uint32_t w, bool re_low, uint32_t (&a_re)[2], uint32_t (&a_im)[2])
{
    const uint32_t hu = (w >> 4) & 0x0F0F0F0Fu, lu = w & 0x0F0F0F0Fu;
    const uint32_t ru = re_low ? lu : hu, iu = re_low ? hu : lu;
    const uint32_t re = (ru + 0x78787878u) ^ 0x80808080u;    // nibble - 8
    const uint32_t im = (iu + 0x78787878u) ^ 0x80808080u;
    const uint32_t ni = (0x88888888u - iu) ^ 0x80808080u;    // 8 - nibble
    // v_perm selector bytes: 0-3 pick from the second source, 4-7 from the first
    a_re[0] = __builtin_amdgcn_perm(ni, re, 0x05010400u);
    a_re[1] = __builtin_amdgcn_perm(ni, re, 0x07030602u);
    a_im[0] = __builtin_amdgcn_perm(re, im, 0x05010400u);
    a_im[1] = __builtin_amdgcn_perm(re, im, 0x07030602u);
}

typedef row16 bu4;

// 16 inputs i0 .. of a row of which inputs below `end` exist (anything past
// it: the weights there are zero); `before`: inputs of the row that lie
// before `row` (earlier chunks).
template <bool VEC>
__device__ __forceinline__ bu4 load16(const uint8_t *row, int i0, int end, int before)
{
    if (!VEC) return load_row16(row, i0, end, before);
    if (i0 >= end) return bu4{0x88888888u, 0x88888888u, 0x88888888u, 0x88888888u};
    return *reinterpret_cast<const bu4 *>(row + i0);
}

// Two k-steps (16 inputs of the lane's row) into both accumulators.
__device__ __forceinline__ void beam_steps(bv4i &acc_re, bv4i &acc_im, const bu4 x, const uint8_t *lw, int p, int g,
                                           int r, bool re_low)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t r0[2], r1[2], m0[2], m1[2];
        unpack4(x[2 * h], re_low, r0, m0);
        unpack4(x[2 * h + 1], re_low, r1, m1);
        const bv4i ar = {(int)r0[0], (int)r0[1], (int)r1[0], (int)r1[1]};
        const bv4i ai = {(int)m0[0], (int)m0[1], (int)m1[0], (int)m1[1]};
        const bv4i b = *reinterpret_cast<const bv4i *>(lw + (((2 * p + h) * 4 + g) * 16 + r) * 16);
        acc_re = __builtin_amdgcn_mfma_i32_16x16x64_i8(ar, b, acc_re, 0, 0, 0);
        acc_im = __builtin_amdgcn_mfma_i32_16x16x64_i8(ai, b, acc_im, 0, 0, 0);
    }
}

// Every wave's LDS accesses are done, its loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));   // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Loads run PREF pairs of k-steps ahead of the MFMAs that use them
// (register double buffer).  KS = 2: two waves share a row block, each half
// of its inputs, and their sums meet in LDS.
template <bool VEC, bool QUANT, int WAVES, int KS, int PREF>
__global__ __launch_bounds__(64 * WAVES) void beamform(const uint8_t *__restrict__ s, int64_t n_samples, int n,
                                                       int64_t stride, uint32_t re_low,
                                                       const uint8_t *__restrict__ w, int n_beams, int shift,
                                                       int lds_weights, void *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r = lane & 15, g = lane >> 4;
    constexpr int ROW_WAVES = WAVES / KS;
    constexpr int ROWS = 16 * ROW_WAVES;
    const int rw = KS == 1 ? wave : wave % ROW_WAVES, ks = KS == 1 ? 0 : wave / ROW_WAVES;
    const int64_t row_blocks = (n_samples + ROWS - 1) / ROWS;
    const bool one_chunk = n <= BEAM_CHUNK;
    // the weights of one chunk, already in operand order in device memory
    // (arranged on the host, see beam_image), into LDS
    auto load_weights = [&](int chunk, int inputs) {
        const bu4 *wc = reinterpret_cast<const bu4 *>(w + (int64_t)chunk * BEAM_LDS);
        const int words = (inputs + BEAM_PAIR - 1) / BEAM_PAIR * BEAM_PAIR * (BEAM_IN_BYTES / 16);
        constexpr int PER = 8;
        for (int k0 = tid; k0 < words; k0 += PER * 64 * WAVES) {
            bu4 v[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int e = k0 + k * 64 * WAVES;
                if (e < words) v[k] = wc[e];
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int e = k0 + k * 64 * WAVES;
                if (e < words) reinterpret_cast<bu4 *>(lw)[e] = v[k];
            }
        }
    };
    bool loaded = false;
    for (int64_t rb = blockIdx.x; rb < row_blocks; rb += gridDim.x) {
        const int64_t t = rb * ROWS + rw * 16 + r;     // this lane's time row
        const bool row_ok = t < n_samples;
        bv4i acc_re = {0, 0, 0, 0}, acc_im = {0, 0, 0, 0};
        for (int c0 = 0; c0 < n; c0 += BEAM_CHUNK) {
            const int cn = min(BEAM_CHUNK, n - c0);
            const int end = row_ok ? cn : 0;
            const int np_all = (cn + BEAM_PAIR - 1) / BEAM_PAIR;   // pairs of k-steps; this wave's: pb .. np - 1
            const int pb = ks == 0 ? 0 : (np_all + 1) / 2;
            const int np = KS == 2 && ks == 0 ? (np_all + 1) / 2 : np_all;
            const uint8_t *row = s + (row_ok ? t : 0) * stride + c0;
            const bool load = !one_chunk || !loaded;
            if (load) {
                if (!one_chunk && loaded) lds_barrier();   // every wave has read the last chunk
                load_weights(c0 / BEAM_CHUNK, cn);
                loaded = true;
            }
            bu4 cur[PREF], nxt[PREF];
#pragma unroll
            for (int k = 0; k < PREF; ++k) cur[k] = load16<VEC>(row, BEAM_PAIR * (pb + k) + 16 * g, end, c0);
            if (load) lds_barrier();
            for (int p0 = pb; p0 < np; p0 += PREF) {
#pragma unroll
                for (int k = 0; k < PREF; ++k)
                    nxt[k] = load16<VEC>(row, BEAM_PAIR * (p0 + PREF + k) + 16 * g, end, c0);
#pragma unroll
                for (int k = 0; k < PREF; ++k)
                    if (p0 + k < np) beam_steps(acc_re, acc_im, cur[k], lw, p0 + k, g, r, re_low != 0);
#pragma unroll
                for (int k = 0; k < PREF; ++k) cur[k] = nxt[k];
            }
        }
        if constexpr (KS == 2) {
            // behind the weights
            int32_t *mine = reinterpret_cast<int32_t *>(lw + lds_weights) + (rw * 64 + lane) * 8;
            if (ks == 1) {
                *reinterpret_cast<bv4i *>(mine) = acc_re;
                *reinterpret_cast<bv4i *>(mine + 4) = acc_im;
            }
            lds_barrier();
            if (ks == 0) {
                acc_re += *reinterpret_cast<const bv4i *>(mine);
                acc_im += *reinterpret_cast<const bv4i *>(mine + 4);
            }
            lds_barrier();
        }
        // C of a 16 x 16 block: lane holds column (beam) lane % 16, rows
        // 4 (lane / 16) .. + 3 of the wave's 16 time rows
        const int b = lane & 15;
        if (ks == 0 && b < n_beams) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int64_t tt = rb * ROWS + rw * 16 + 4 * g + k;
                if (tt >= n_samples) continue;
                const int64_t o = (tt * n_beams + b) * 2;
                if (QUANT) {
                    // divide by 2^shift, rounded half to even, clipped to [-127, 127]
                    int32_t v2[2] = {acc_re[k], acc_im[k]};
                    int8_t q[2];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        int64_t v = v2[u];
                        if (shift > 0) v = (v + (INT64_C(1) << (shift - 1)) - 1 + ((v >> shift) & 1)) >> shift;
                        q[u] = (int8_t)(v < -127 ? -127 : (v > 127 ? 127 : v));
                    }
                    int8_t *po = reinterpret_cast<int8_t *>(out) + o;
                    po[0] = q[0];
                    po[1] = q[1];
                } else {
                    int32_t *po = reinterpret_cast<int32_t *>(out) + o;
                    po[0] = acc_re[k];
                    po[1] = acc_im[k];
                }
            }
        }
    }
}

// Operand-order image of the weights (host): nchunks x BEAM_LDS bytes, the
// LDS contents of each chunk of BEAM_CHUNK inputs as the kernel expects them.
// Input i of a chunk, beam b: step s = 2 (i / 64) + (i % 16) / 8, lane group
// (i % 64) / 16; byte offset ((4 s + group) * 16 + b) * 16 + 2 (i % 8) holds
// (Re w, Im w).  Inputs past N and beams past n_beams are zero.
int64_t beam_image_bytes(int n) { return (int64_t)((n + BEAM_CHUNK - 1) / BEAM_CHUNK) * BEAM_LDS; }

void beam_image(const int8_t *w, int n, int n_beams, uint8_t *img)
{
    const int nchunks = (n + BEAM_CHUNK - 1) / BEAM_CHUNK;
    for (int c = 0; c < nchunks; ++c) {
        uint8_t *base = img + (int64_t)c * BEAM_LDS;
        for (int i = 0; i < BEAM_CHUNK; ++i) {
            const int gi = c * BEAM_CHUNK + i;
            const int step = 2 * (i / 64) + (i % 16) / 8, grp = (i % 64) / 16;
            for (int b = 0; b < BEAMS_MAX; ++b) {
                int wr = 0, wi = 0;
                if (gi < n && b < n_beams) {
                    wr = w[((int64_t)b * n + gi) * 2];
                    wi = w[((int64_t)b * n + gi) * 2 + 1];
                }
                uint8_t *o = base + ((step * 4 + grp) * 16 + b) * 16 + 2 * (i % 8);
                o[0] = (uint8_t)(int8_t)wr;
                o[1] = (uint8_t)(int8_t)wi;
            }
        }
    }
}

namespace {

template <bool VEC, bool QUANT, int WAVES, int KS, int PREF>
hipError_t launch_waves(const uint8_t *s, int64_t n_samples, int n, int64_t stride, uint32_t re_low,
                        const uint8_t *d_w, int n_beams, int shift, void *out, int cus, hipStream_t stream)
{
    constexpr int ROWS = 16 * WAVES / KS;
    const int inputs = n < BEAM_CHUNK ? (n + BEAM_PAIR - 1) / BEAM_PAIR * BEAM_PAIR : BEAM_CHUNK;
    const int lds = inputs * BEAM_IN_BYTES;
    // resident workgroups of a CU, by LDS (160 KiB, the sums of KS = 2
    // included) and by four waves per SIMD
    const int all = lds + (KS == 2 ? ROWS / 16 * 64 * 32 : 0);
    const int by_lds = 160 * 1024 / all, by_waves = 16 / WAVES;
    const int64_t slots = (int64_t)cus * (by_lds < by_waves ? by_lds : by_waves);
    const int64_t blocks = (n_samples + ROWS - 1) / ROWS;
    hipLaunchKernelGGL((beamform<VEC, QUANT, WAVES, KS, PREF>), dim3((unsigned)(blocks < slots ? blocks : slots)),
                       dim3(64 * WAVES), all, stream, s, n_samples, n, stride, re_low, d_w, n_beams, shift, lds, out);
    return hipGetLastError();
}

// Enough rows for six waves of 16 on every compute unit (T from 96 per
// unit up): each wave its own rows, two pairs of k-steps ahead -- N = 2048, T =
// 32768: 13.8 us (eight pairs ahead 17.0, rows shared by two waves 15.6).
// Fewer: two waves per row block, four pairs ahead, and below 32 rows per
// unit half as many rows per workgroup -- N = 2048, T = 4096: 7.3 us (own
// rows 10.5); N = 1000, T = 16384: 7.2 us (own rows 8.5).
template <bool VEC, bool QUANT>
hipError_t launch_rows(const uint8_t *s, int64_t n_samples, int n, int64_t stride, uint32_t re_low, const uint8_t *d_w,
                       int n_beams, int shift, void *out, int cus, hipStream_t stream)
{
    if (n_samples >= 96 * (int64_t)cus)
        return launch_waves<VEC, QUANT, 4, 1, 2>(s, n_samples, n, stride, re_low, d_w, n_beams, shift, out, cus, stream);
    if (n_samples > 32 * (int64_t)cus)
        return launch_waves<VEC, QUANT, 8, 2, 4>(s, n_samples, n, stride, re_low, d_w, n_beams, shift, out, cus, stream);
    return launch_waves<VEC, QUANT, 4, 2, 4>(s, n_samples, n, stride, re_low, d_w, n_beams, shift, out, cus, stream);
}

}  // namespace

// Once per device, before any launch: with the shared sums the instances of
// KS = 2 may pass the default dynamic-LDS limit.
hipError_t init_beam_kernel()
{
    hipError_t e = hipSuccess;
    for (const void *f : {(const void *)beamform<true, true, 8, 2, 4>, (const void *)beamform<true, false, 8, 2, 4>,
                          (const void *)beamform<false, true, 8, 2, 4>, (const void *)beamform<false, false, 8, 2, 4>,
                          (const void *)beamform<true, true, 4, 2, 4>, (const void *)beamform<true, false, 4, 2, 4>,
                          (const void *)beamform<false, true, 4, 2, 4>, (const void *)beamform<false, false, 4, 2, 4>})
        if (e == hipSuccess)
            e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, BEAM_LDS + 8192);
    return e;
}

// `cus`: compute units of the device.
hipError_t launch_beamform(const uint8_t *s, int64_t n_samples, int n, int64_t stride, uint32_t re_low,
                           const int8_t *d_w, int n_beams, int shift, void *out, int cus, hipStream_t stream)
{
    if (n_samples <= 0) return hipSuccess;
    const bool vec = (reinterpret_cast<uintptr_t>(s) % 16) == 0 && stride % 16 == 0 && n % 16 == 0;
    const bool quant = shift >= 0;
    const uint8_t *w = reinterpret_cast<const uint8_t *>(d_w);
    if (vec && quant) return launch_rows<true, true>(s, n_samples, n, stride, re_low, w, n_beams, shift, out, cus, stream);
    if (vec) return launch_rows<true, false>(s, n_samples, n, stride, re_low, w, n_beams, shift, out, cus, stream);
    if (quant) return launch_rows<false, true>(s, n_samples, n, stride, re_low, w, n_beams, shift, out, cus, stream);
    return launch_rows<false, false>(s, n_samples, n, stride, re_low, w, n_beams, shift, out, cus, stream);
}

}  // namespace xeng
