// bf16 PCONV on the matrix cores, main kernel: Eq. (1) as nine shifted contractions over flat pixels.
//
// Y[f, p] += sum_c W_rs[f, c] * X[c, p shifted by (r, s)] for every tap (r, s), dense over the masked
// weights (v_mfma_f32_32x32x16_bf16, fp32 accumulation); a (tap, 16 channels, 32 filters) block
// without a kept weight is skipped.
//
// Work decomposition.  The output pixels of the whole batch are one flat list; a workgroup owns a run
// of it and MB blocks of 32 filters.  Its waves are WP pixel parts x WK channel parts: a wave holds
// MB x NB blocks of 32 filters x 32 pixels and walks every WK-th block of 16 input channels (the WK
// partial sums are added through LDS at the end, in a fixed order).  A flat run has no ragged tile
// edges: 49-pixel images fill the instruction as well as large ones.
//
// Staging.  The taps of a run of pixels read, in every image it touches, one contiguous range of each
// channel plane (from the first tap of the first pixel to the last tap of the last).  That range is
// staged for 16 channels at a time as two planes of [pixel][8 channels], so that a lane's operand is
// one 128-bit read.  One staging item is 8 pixels x 8 channels: eight 16-byte loads, for NCHW an 8x8
// transpose in registers (32 v_perm), eight 16-byte LDS writes.  The loads of the next block are in
// flight during the matrix instructions of the present one, and two LDS buffers are used in turn (one
// barrier per block; none at all with WP = 1, where every wave reads only what it staged itself).
// After every eight pixels one 16-byte slot is left free: the LDS writes of neighbouring lanes, which
// are eight pixels apart, would otherwise all fall on the same banks.  A lane's nine tap addresses do
// not change from block to block and are kept in registers; a tap outside the image reads a slot of
// zeros, so the inner loop has no bounds arithmetic.
//
// What bounds it: at full occupancy the vector-memory pipe (18 KB of weight fragments per wave, two
// blocks of filters and 16 channels, for 36 matrix instructions) and the fixed start and end of a
// workgroup (some 7000 cycles before the first matrix instruction, 2500 to 5000 after the last); with
// few workgroups the latency of one workgroup's chain of channel blocks.  Counters, 32 images 256@14: the
// matrix units are busy 17 % of the time, a wave waits for data 40 % of it and to issue 27 %.  Measured
// on one MI355X, the seven ResNet-50 3x3 shapes, NCHW, in us, calls back to back in a graph, against the
// tiled-image kernel of pconv_mfma.hip:
//   one image    64@56 5.2 (9.3)   128@56/2 9.0 (13.3)  128@28 5.4 (12.7)  256@28/2 10.8 (20.6)
//                256@14 7.2 (20.3)  512@14/2 10.3 (35.2)  512@7 13.1 (37.6)
//   32 images    64@56 18.7 (37.9)  128@56/2 29.3 (37.8)  128@28 16.6 (31.1)  256@28/2 28.9 (30.1)
//                256@14 16.0 (27.5)  512@14/2 30.7 (47.3)  512@7 25.0 (38.3)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <string>
#include <type_traits>

#include "pconv_internal.h"

namespace pconv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// n / d for n < 2^31 by one multiplication: Granlund and Montgomery's division by an invariant, with the
// multiplier floor(2^32 (2^s - d) / d) + 1 and s = ceil(log2 d)
struct FastDiv { uint32_t mul, shift; };
FastDiv make_fast_div(uint32_t d)
{
    uint32_t s = 0;
    while ((uint64_t(1) << s) < d) ++s;
    return {uint32_t(((uint64_t(1) << 32) * ((uint64_t(1) << s) - d)) / d + 1), s};
}
__device__ __forceinline__ int fast_div(int n, FastDiv d)
{
    return int((__umulhi(uint32_t(n), d.mul) + uint32_t(n)) >> d.shift);
}

struct FlatArgs {
    const uint16_t *x; uint16_t *y; const float *bias;
    const uint16_t *wd;             // [fblocks][cb16][9][32][16] bf16 bit patterns
    const uint32_t *nz;             // [cb16 / 2][fblocks]: bit (2 * tap + half)
    int c_in, w, c_out, hw, wo, howo, h;
    int stride, relu;
    int cb16, fblocks;              // blocks of 16 channels that hold any, blocks of 32 filters
    int wd_cb16;                    // blocks of 16 channels in a row of wd (even)
    int total;                      // output pixels of the batch
    int rhw;                        // h * w rounded up to 8
    FastDiv div_howo, div_wo, div_rhw;
    int wp_log2, wk;
    int bias_at;                    // where the bias lies in LDS, in floats
    int plane;                      // 16-byte slots of a staged plane
    int tiles, fgroups, filter_major;
};

// 16 bytes from an address that need not be aligned to more than an element
__device__ __forceinline__ u32x4 load16(const char *p)
{
    u32x4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

template <int LAYOUT, int MB, int NB, int R>
__global__ void __launch_bounds__(512)
conv_flat_kernel(const FlatArgs a)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 slots[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wp = 1 << a.wp_log2, wpi = wave & (wp - 1), wki = wave >> a.wp_log2;
    const int col = lane & 31, kg = lane >> 5;

    // Workgroups whose ids are equal mod 8 run on one XCD (one L2): each gets a contiguous eighth of
    // the (tile, filter group) pairs, ordered so that neighbours share the larger of the two operands.
    const int pairs = a.tiles * a.fgroups;
    const int u = int(blockIdx.x & 7) * ((pairs + 7) >> 3) + int(blockIdx.x >> 3);
    if (u >= pairs || int(blockIdx.x >> 3) >= ((pairs + 7) >> 3)) return;
    const int tile = a.filter_major ? u % a.tiles : u / a.fgroups;
    const int fg = a.filter_major ? u / a.tiles : u % a.fgroups;

    // ---- the run of output pixels and the input ranges it reads ----
    const int p0 = tile * (NB * 32 << a.wp_log2);
    const int p_end = min(p0 + (NB * 32 << a.wp_log2), a.total);
    const int img0 = fast_div(p0, a.div_howo), img_last = fast_div(p_end - 1, a.div_howo);
    auto centre = [&](int r) { const int oy = fast_div(r, a.div_wo); return (oy * a.w + (r - oy * a.wo)) * a.stride; };
    const int lo0 = max(0, min(centre(p0 - img0 * a.howo) - a.w - 1, a.hw - 8)) & ~7;
    const int hi_last = min(a.hw, centre(p_end - 1 - img_last * a.howo) + a.w + 2);
    const int base1 = ((img_last == img0 ? hi_last : a.hw) - lo0 + 7) & ~7;      // staged position of the second image
    const int staged = img_last == img0 ? base1 : base1 + (img_last - img0 - 1) * a.rhw + ((hi_last + 7) & ~7);

    // ---- what this thread stages, the same for every block of channels ----
    const int tid_g = int(threadIdx.x) & ((64 << a.wp_log2) - 1);               // thread within the channel part
    const int g_item = tid_g & 1;                                              // which plane of 8 channels
    uint32_t src[R];                                                           // byte offset of the item's first element
    int dst[R], dst_step[R];                                                   // slot of its first pixel (-1: no item); pixel at which a free slot is stepped over
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int pos = ((tid_g >> 1) + i * (32 << a.wp_log2)) * 8;
        const bool ok = pos < staged;
        int img = img0, q = lo0 + pos;
        if (pos >= base1) {
            const int t = pos - base1, s = fast_div(t, a.div_rhw);
            img = img0 + 1 + s; q = t - s * a.rhw;
        }
        // the last item of a plane is moved back to end with it (and writes some pixels a second time)
        const int q8 = min(q, a.hw - 8), wpos = pos - (q - q8);
        const uint32_t e = LAYOUT == PCONV_NCHW ? uint32_t(img * a.c_in * a.hw + q8)
                                                : uint32_t((img * a.hw + q8) * a.c_in);
        src[i] = ok ? e * 2u : 0u;
        dst[i] = ok ? g_item * a.plane + wpos + (wpos >> 3) : -1;
        dst_step[i] = 8 - (wpos & 7);
    }
    const char *xb = reinterpret_cast<const char *>(a.x);
    const uint32_t plane_step = uint32_t(a.hw) * 2u, item_step = (LAYOUT == PCONV_NCHW ? plane_step : 2u) * 8u * uint32_t(g_item);
    auto load_block = [&](int cb, u32x4 (&raw)[R][8]) {
        const int c0 = cb * 16;
        if (c0 + 16 <= a.c_in) {                                               // (uniform)
            const char *base = xb + (LAYOUT == PCONV_NCHW ? uint32_t(c0) * plane_step : uint32_t(c0) * 2u);
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    raw[i][j] = load16(base + (LAYOUT == PCONV_NCHW ? uint32_t(j) * plane_step : uint32_t(j * a.c_in) * 2u) + (src[i] + item_step));
        } else {
            // the last, partial block: a channel beyond c_in reads the last one and is zeroed below
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int c = LAYOUT == PCONV_NCHW ? min(c0 + g_item * 8 + j, a.c_in - 1) : min(c0 + g_item * 8, a.c_in - 8);
                    raw[i][j] = load16(xb + (LAYOUT == PCONV_NCHW ? uint32_t(c) * plane_step : uint32_t(c + j * a.c_in) * 2u) + src[i]);
                }
        }
    };
    const int buf_slots = a.wk * 2 * a.plane + 1;                              // the last slot of a buffer holds zeros
    auto store_block = [&](int cb, int buf, u32x4 (&raw)[R][8]) {
        if (cb * 16 + 16 > a.c_in) {                                           // (uniform)
            const int left = a.c_in - cb * 16 - g_item * 8;                    // channels of the item that exist
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if ((LAYOUT == PCONV_NCHW ? j : 0) >= left) raw[i][j] = u32x4{0u, 0u, 0u, 0u};   // (NHWC: c_in is a multiple of 8)
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (dst[i] < 0) continue;
            u32x4 *lp = slots + buf * buf_slots + wki * 2 * a.plane + dst[i];
            u32x4 *lp1 = lp + 1;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                u32x4 v;
                if (LAYOUT == PCONV_NCHW) {
                    // pixel j: 16-bit half j % 2 of dword j / 2 of the eight channel rows
                    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_perm(raw[i][2 * k + 1][j >> 1], raw[i][2 * k][j >> 1], sel);
                } else {
                    v = raw[i][j];
                }
                (j >= dst_step[i] ? lp1 : lp)[j] = v;
            }
        }
    };

    // ---- weights: a wave's fragments of a block of channels are 9 KB in a row per block of filters ----
    int fb[MB];                      // (a block beyond the last one repeats it; its sums are not stored)
#pragma unroll
    for (int m = 0; m < MB; ++m) fb[m] = min(fg * MB + m, a.fblocks - 1);
    // a window of kWin taps ahead of the one in use: a fragment that has been used is replaced at once
    // by the one kWin places later, which may belong to the next block of channels
    constexpr int kWin = MB * NB == 4 && MB == 2 ? 3 : 9;
    u32x4 wf[kWin][MB];
    auto load_weight = [&](int cb, int q, int m) {
        const uint32_t e = (uint32_t(fb[m] * a.wd_cb16 + cb) * 9u + uint32_t(q)) * 512u;
        wf[q % kWin][m] = *reinterpret_cast<const u32x4 *>(a.wd + e + uint32_t(lane & 31) * 16u + uint32_t(kg) * 8u);
    };

    u32x4 raw[R][8];
    const int iters = (a.cb16 + a.wk - 1) / a.wk;
    {
        const int cb = min(wki, a.cb16 - 1);
        load_block(cb, raw);
#pragma unroll
        for (int q = 0; q < kWin; ++q)
#pragma unroll
            for (int m = 0; m < MB; ++m) load_weight(cb, q, m);
    }

    // ---- this lane's tap addresses (bytes, in buffer 0) ----
    int addr[9][NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int p = p0 + (wpi * NB + j) * 32 + col;
        const int img = fast_div(min(p, a.total - 1), a.div_howo), r = min(p, a.total - 1) - img * a.howo;
        const int oy = fast_div(r, a.div_wo), ox = r - oy * a.wo;
        const int iy = oy * a.stride, ix = ox * a.stride;
        const int pos = (img == img0 ? -lo0 : base1 + (img - img0 - 1) * a.rhw) + iy * a.w + ix;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int dy = q / 3 - 1, dx = q % 3 - 1;
            // (a negative coordinate is a large unsigned one; no short-circuits: selects, not branches)
            const bool ok = (p < p_end) & (uint32_t(iy + dy) < uint32_t(a.h)) & (uint32_t(ix + dx) < uint32_t(a.w));
            const int t = pos + dy * a.w + dx;
            addr[q][j] = (ok ? (wki * 2 + kg) * a.plane + t + (t >> 3) : buf_slots - 1) * 16;
        }
    }

    f32x16 acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[m][j] = 0.0f;

    // bias of the workgroup's filters, behind everything else in LDS (-0 where there is none: x + -0 = x)
    float *bias_lds = reinterpret_cast<float *>(slots) + a.bias_at;
    if (int(threadIdx.x) < MB * 32) {
        const int f = fg * MB * 32 + int(threadIdx.x);
        bias_lds[threadIdx.x] = a.bias && f < a.c_out ? a.bias[f] : -0.0f;
    }
    if (threadIdx.x < 2) slots[threadIdx.x * buf_slots + buf_slots - 1] = u32x4{0u, 0u, 0u, 0u};
    store_block(min(wki, a.cb16 - 1), 0, raw);
    __syncthreads();

    // NCHW: pixels are the rows of the instruction's result and filters its columns, so that a lane
    // ends up with four consecutive pixels of one filter; NHWC: the other way round.
    auto mfma = [&](const u32x4 &w, const bf16x8 &x, const f32x16 &c) {
        const bf16x8 wv = __builtin_bit_cast(bf16x8, w);
        return LAYOUT == PCONV_NCHW ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, wv, c, 0, 0, 0)
                                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, x, c, 0, 0, 0);
    };
    const char *lds_bytes = reinterpret_cast<const char *>(slots);
    // (constant address space: scalar loads, which the waits for vector loads do not involve)
    typedef const uint32_t __attribute__((address_space(4))) *ConstWords;
    const ConstWords nz = reinterpret_cast<ConstWords>(reinterpret_cast<uintptr_t>(a.nz));
    auto block_bits = [&](int cb, int m) -> uint32_t { return nz[(cb >> 1) * a.fblocks + fb[m]] >> (cb & 1); };
    uint32_t bits[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) bits[m] = block_bits(min(wki, a.cb16 - 1), m);

    auto step = [&](int it, auto more_c) {
        constexpr bool MORE = decltype(more_c)::value;
        const int cb = it * a.wk + wki;
        const int next = min(cb + a.wk, a.cb16 - 1);
        const int buf = it & 1;
        uint32_t next_bits[MB];
        if (MORE) {
            load_block(next, raw);
#pragma unroll
            for (int m = 0; m < MB; ++m) next_bits[m] = block_bits(next, m);
        }
        auto replace_weight = [&](int q, int m) {
            if (q + kWin < 9) load_weight(min(cb, a.cb16 - 1), q + kWin, m);
            else if (MORE) load_weight(next, q + kWin - 9, m);
        };
        const char *bp = lds_bytes + buf * buf_slots * 16;
        bool full = cb < a.cb16;
#pragma unroll
        for (int m = 0; m < MB; ++m) full = full && (bits[m] & 0x15555u) == 0x15555u;
        if (full) {
            constexpr int AHEAD = MB * NB <= 2 ? 2 : 1;  // taps by which the pixel fragments are read ahead (registers permitting)
            bf16x8 xv[AHEAD + 1][NB];
#pragma unroll
            for (int q = 0; q < AHEAD; ++q)
#pragma unroll
                for (int j = 0; j < NB; ++j) xv[q][j] = *reinterpret_cast<const bf16x8 *>(bp + addr[q][j]);
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                if (q + AHEAD < 9) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) xv[(q + AHEAD) % (AHEAD + 1)][j] = *reinterpret_cast<const bf16x8 *>(bp + addr[q + AHEAD][j]);
                }
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int j = 0; j < NB; ++j) acc[m][j] = mfma(wf[q % kWin][m], xv[q % (AHEAD + 1)][j], acc[m][j]);
#pragma unroll
                for (int m = 0; m < MB; ++m) replace_weight(q, m);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    if (cb < a.cb16 && ((bits[m] >> (2 * q)) & 1u)) {
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            acc[m][j] = mfma(wf[q % kWin][m], *reinterpret_cast<const bf16x8 *>(bp + addr[q][j]), acc[m][j]);
                    }
                    replace_weight(q, m);
                }
            }
        }
        if (MORE) {
            store_block(next, buf ^ 1, raw);
#pragma unroll
            for (int m = 0; m < MB; ++m) bits[m] = next_bits[m];
            if (a.wp_log2) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
        }
    };
    for (int it = 0; it + 1 < iters; ++it) step(it, std::true_type{});
    step(iters - 1, std::false_type{});

    // ---- epilogue ----
    // All sums go to LDS (over the staging buffers) as the instruction leaves them: four consecutive
    // pixels (NHWC: filters) of one filter (pixel) per lane and group.  They are read back so that
    // eight neighbouring lanes hold neighbouring octets, the channel parts are added in order, and
    // bias, ReLU and rounding give 16 bytes per lane, which makes whole cache lines per store (the
    // four values a lane starts with would be stored as 8 bytes here and there).
    constexpr int G = MB * NB * 4, kGroupPitch = 65;                           // (one slot more than lanes: bank spread)
    constexpr int OCT = LAYOUT == PCONV_NCHW ? NB * 4 : MB * 4;                // octets in a row
    f32x4 *red = reinterpret_cast<f32x4 *>(slots);
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                red[(wave * G + (m * NB + j) * 4 + g) * kGroupPitch + lane] =
                    f32x4{acc[m][j][4 * g], acc[m][j][4 * g + 1], acc[m][j][4 * g + 2], acc[m][j][4 * g + 3]};
    __syncthreads();
#pragma unroll 2
    for (int id = wki * 64 + lane; id < MB * NB * 128; id += a.wk * 64) {
        const int o = id & (OCT - 1), c = (id / OCT) & 31, outer = id / (OCT * 32);
        const int m = LAYOUT == PCONV_NCHW ? outer : o >> 2, j = LAYOUT == PCONV_NCHW ? o >> 2 : outer;
        const f32x4 *rp = red + (wpi * G + (m * NB + j) * 4 + (o & 3)) * kGroupPitch + c;
        f32x4 v0 = rp[0], v1 = rp[32];
        for (int k = 1; k < a.wk; ++k) {
            rp += (G * kGroupPitch) << a.wp_log2;
            v0 += rp[0]; v1 += rp[32];
        }
        union { __bf16 e[8]; uint16_t u[8]; u32x4 d; } out;
        const int f = (fg * MB + m) * 32 + (LAYOUT == PCONV_NCHW ? c : 8 * (o & 3));
        const int p = p0 + (wpi * NB + j) * 32 + (LAYOUT == PCONV_NCHW ? 8 * (o & 3) : c);
        const float *bp = bias_lds + m * 32 + (LAYOUT == PCONV_NCHW ? c : 8 * (o & 3));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float t = (k < 4 ? v0[k & 3] : v1[k & 3]) + bp[LAYOUT == PCONV_NCHW ? 0 : k];
            out.e[k] = __bf16(a.relu ? fmaxf(t, 0.0f) : t);
        }
        if ((f >= a.c_out) | (p >= p_end)) continue;
        if (LAYOUT == PCONV_NCHW) {
            const int img = fast_div(p, a.div_howo), r = p - img * a.howo;
            if ((r + 8 <= a.howo) & (p + 8 <= p_end)) {
                __builtin_memcpy(a.y + (uint32_t(img * a.c_out + f) * uint32_t(a.howo) + uint32_t(r)), &out.d, 16);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int im = fast_div(p + k, a.div_howo);
                    if (p + k < p_end) a.y[uint32_t(im * a.c_out + f) * uint32_t(a.howo) + uint32_t(p + k - im * a.howo)] = out.u[k];
                }
            }
        } else {
            uint16_t *yp = a.y + (uint32_t(p) * uint32_t(a.c_out) + uint32_t(f));
            if (f + 8 <= a.c_out) {
                __builtin_memcpy(yp, &out.d, 16);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (f + k < a.c_out) yp[k] = out.u[k];
            }
        }
    }
}

// Upper bound of the staged pixels of any run of np output pixels (see the kernel's `staged`).
int64_t staged_bound(int np, int64_t hw, int64_t howo, int64_t w, int64_t wo, int stride)
{
    const int64_t rhw = (hw + 7) & ~int64_t(7);
    // distance of the first and last centre of k pixels of one image (stride 2: line ends skip an input line)
    auto centres = [&](int64_t k) { return stride == 1 ? k - 1 : 2 * (k - 1) + ((k - 1) / wo + 1) * (2 * w - 2 * wo); };
    int64_t most = std::min(rhw, (centres(std::min<int64_t>(np, howo)) + 2 * w + 3 + 21) & ~int64_t(7));
    for (int64_t images = 2; images <= (np - 2) / howo + 2 && images <= np; ++images) {
        // the first image from its first tap to its end, the last one from its start to the last tap
        const int64_t ends = np - (images - 2) * howo;
        const int64_t both = centres(ends) + 2 * w + 3 + (stride == 1 ? 0 : 3 * w - 2 * wo + 1) + 28;
        most = std::max(most, (images - 2) * rhw + std::min(2 * rhw, both & ~int64_t(7)));
    }
    return most;
}

constexpr int64_t kLdsOfUnit = 160 * 1024;

template <int LAYOUT, int MB, int NB, int R>
hipError_t launch_flat(const FlatArgs &a, dim3 grid, dim3 block, int64_t lds, hipStream_t st, int dev)
{
    // More dynamic LDS than the default limit: raised once per device (the flag is set to the same
    // value by every thread that gets here first).
    static std::atomic<bool> attr_done[64];
    if (dev < 0 || dev >= 64 || !attr_done[dev].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_flat_kernel<LAYOUT, MB, NB, R>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsOfUnit));
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_done[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((conv_flat_kernel<LAYOUT, MB, NB, R>), grid, block, size_t(lds), st, a);
    return hipGetLastError();
}

// Launch shape: MB x NB blocks of 32 filters x 32 pixels per wave, WP pixel parts x WK channel parts.
struct FlatShape { int index, mb, nb, wp, wk, r; int64_t plane, lds; };

constexpr int kShapes[][4] = {{2, 2, 4, 1}, {2, 2, 2, 1}, {2, 2, 2, 2}, {2, 2, 1, 4}, {2, 1, 4, 1}, {2, 1, 2, 2},
                              {1, 2, 4, 1}, {1, 2, 2, 2}, {1, 2, 1, 4}, {1, 1, 4, 1}, {1, 1, 2, 2}, {1, 1, 2, 4}, {1, 1, 1, 8}};
constexpr int kNumShapes = int(sizeof kShapes / sizeof kShapes[0]);
std::atomic<int> g_force_shape{-1};      // test override, see set_flat_shape

// The shape with the smallest estimate of the layer's time, in microseconds; false if the kernel does
// not serve the call.  Few workgroups: the time of one, a start and end and per block of channels the
// latency of its loads and LDS traffic.  Many: what a compute unit spends on a workgroup, per wave and
// block of outputs, and per wave and block of channels for every block of weights, of matrix
// instructions and for 64 staging items.  The constants are a fit to all shapes on thirteen layers (24
// to 512 channels, 7 to 224 pixels square, both strides) with 1 to 32 images: the shape chosen takes
// 1 % longer than the fastest one on average, 20 % at most (512@7, 32 images: {1, 2, 1, 4} takes 25.0 us,
// {2, 2, 1, 4} 21.9).
bool choose_flat(const pconv_handle *h, int n, int hin, int win, int stride, int layout, FlatShape &best)
{
    const int hw = hin * win, wo = (win - 1) / stride + 1, howo = ((hin - 1) / stride + 1) * wo, total = n * howo;
    const int cb16 = (h->c_in + 15) / 16, wd_cb16 = (h->c_in + 31) / 32 * 2, fblocks = (h->c_out + 31) / 32;
    // (a staging item is eight pixels of a plane; NHWC pixels are read in whole octets of channels)
    if (hw < 8 || (layout == PCONV_NHWC && h->c_in % 8 != 0)) return false;
    if (int64_t(fblocks) * wd_cb16 * 9 * 512 >= (int64_t(1) << 31)) return false;   // (32-bit weight offsets)
    best = FlatShape{};
    double best_time = 0.0;
    const int cus = h->cus > 0 ? h->cus : 256, forced = g_force_shape.load();
    for (int k = 0; k < kNumShapes; ++k) {
        const auto &c = kShapes[k];
        FlatShape s{k, c[0], c[1], c[2], c[3], 1, 0, 0};
        if (forced >= 0 && k != forced) continue;
        if (s.mb > fblocks || s.wk > cb16) continue;
        const int np = 32 * s.nb * s.wp, waves = s.wp * s.wk;
        const int64_t bound = staged_bound(np, hw, howo, win, wo, stride);
        s.plane = bound + bound / 8;
        s.lds = std::max<int64_t>(2 * (s.wk * 2 * s.plane + 1) * 16, int64_t(waves) * s.mb * s.nb * 4 * 65 * 16) + 256;
        const int64_t items = bound / 4;
        s.r = items <= 64 * s.wp ? 1 : 2;
        if (items > 64 * s.wp * s.r || (s.r == 2 && (s.mb == 2 || layout == PCONV_NHWC)) || s.lds > kLdsOfUnit) continue;
        const int iters = (cb16 + s.wk - 1) / s.wk;
        const int64_t tiles = (total + np - 1) / np, fgroups = (fblocks + s.mb - 1) / s.mb;
        const double groups = double(tiles) * fgroups / cus;
        const double share = double(items) / (64 * s.wp);
        const double chain = 2.4 + iters * ((s.mb == 1 ? 1.33 : s.nb == 1 ? 1.44 : 1.99) + 0.1 * share);
        const double busy = waves * (0.064 * s.mb * s.nb + iters * (0.04 * s.mb + 0.1 * s.mb * s.nb + 0.04 * share));
        const int resident = int(std::min<int64_t>(kLdsOfUnit / s.lds, 8 / waves));
        const double rounds = std::ceil(groups / resident);
        const double lo = std::min(groups * busy, rounds * chain), hi = std::max(groups * busy, rounds * chain);
        const double time = hi + 0.25 * lo;
        if (best.mb == 0 || time < best_time) { best = s; best_time = time; }
    }
    if (best.mb == 0) return false;
    const int np = 32 * best.nb * best.wp;
    return int64_t((total + np - 1) / np) * ((fblocks + best.mb - 1) / best.mb) <= 0x3FFFFFFF;
}

}  // namespace

void set_flat_shape(int index) { g_force_shape.store(index >= 0 && index < kNumShapes ? index : -1); }

int flat_shape_of(const pconv_handle *h, int n, int hin, int win, int stride, int layout)
{
    FlatShape s;
    return choose_flat(h, n, hin, win, stride, layout, s) ? s.index : -1;
}

bool launch_conv_flat(const pconv_handle *h, const void *x, void *y, const float *bias, int n, int hin, int win,
                      int stride, int layout, int relu, void *stream, int &rc)
{
    FlatShape best;
    if (!choose_flat(h, n, hin, win, stride, layout, best)) return false;
    FlatArgs a;
    a.x = static_cast<const uint16_t *>(x); a.y = static_cast<uint16_t *>(y); a.bias = bias;
    a.wd = h->d_wdense; a.nz = h->d_wnz;
    a.c_in = h->c_in; a.h = hin; a.w = win; a.c_out = h->c_out;
    const int ho = (hin - 1) / stride + 1;
    a.wo = (win - 1) / stride + 1; a.hw = hin * win; a.howo = ho * a.wo;
    a.stride = stride; a.relu = relu;
    a.cb16 = (h->c_in + 15) / 16; a.wd_cb16 = (h->c_in + 31) / 32 * 2; a.fblocks = (h->c_out + 31) / 32;
    a.total = n * a.howo;
    a.rhw = (a.hw + 7) & ~7;
    a.div_howo = make_fast_div(uint32_t(a.howo)); a.div_wo = make_fast_div(uint32_t(a.wo));
    a.div_rhw = make_fast_div(uint32_t(a.rhw));
    const int mb = best.mb, nb = best.nb, wp = best.wp, wk = best.wk, r = best.r;
    const int np = 32 * nb * wp;
    const int64_t lds = best.lds, plane = best.plane;
    a.bias_at = int((lds - 256) / 4);
    a.wp_log2 = wp == 4 ? 2 : wp == 2 ? 1 : 0; a.wk = wk; a.plane = int(plane);
    a.tiles = (a.total + np - 1) / np; a.fgroups = (a.fblocks + mb - 1) / mb;
    a.filter_major = int64_t(h->c_out) * 9 > int64_t(n) * a.hw;
    const int64_t pairs = int64_t(a.tiles) * a.fgroups;
    const dim3 grid{unsigned((pairs + 7) / 8 * 8)}, block{unsigned(64 * wp * wk)};
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto pick = [&](auto lay, auto rr) {
        constexpr int L = decltype(lay)::value, RR = decltype(rr)::value;
        if constexpr (RR == 1) {
            if (mb == 2 && nb == 2) return launch_flat<L, 2, 2, RR>(a, grid, block, lds, st, h->device);
            if (mb == 2 && nb == 1) return launch_flat<L, 2, 1, RR>(a, grid, block, lds, st, h->device);
        }
        if (mb == 1 && nb == 2) return launch_flat<L, 1, 2, RR>(a, grid, block, lds, st, h->device);
        return launch_flat<L, 1, 1, RR>(a, grid, block, lds, st, h->device);
    };
    using std::integral_constant;
    hipError_t e;
    if (layout == PCONV_NHWC) e = pick(integral_constant<int, PCONV_NHWC>{}, integral_constant<int, 1>{});
    else if (r == 1) e = pick(integral_constant<int, PCONV_NCHW>{}, integral_constant<int, 1>{});
    else e = pick(integral_constant<int, PCONV_NCHW>{}, integral_constant<int, 2>{});
    rc = PCONV_OK;
    if (e != hipSuccess) {
        set_error(std::string("pconv_conv2d (matrix-core kernel): ") + hipGetErrorName(e));
        rc = PCONV_HIP_ERROR;
    }
    return true;
}

}  // namespace pconv
