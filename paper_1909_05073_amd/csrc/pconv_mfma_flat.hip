// bf16 PCONV on the matrix cores, main kernel: Eq. (1) as nine shifted contractions over flat pixels.
//
// Y[f, p] += sum_c W_rs[f, c] * X[c, p shifted by (r, s)] for every tap (r, s), dense over the masked
// weights (v_mfma_f32_32x32x16_bf16, fp32 accumulation); a (tap, 16 channels, 32 filters) block
// without a kept weight is skipped.
//
// Work decomposition.  The output pixels of the whole batch are one flat list; a workgroup owns a run
// of it and a group of filters.  Its waves are WP pixel parts x WF filter parts x WK channel parts: a wave
// holds MB x NB blocks of 32 filters x 32 pixels and walks every WK-th step of KB blocks of 16 input
// channels (the WK partial sums are added through LDS at the end, in a fixed order).  A flat run has no
// ragged tile edges: 49-pixel images fill the instruction as well as large ones.
//
// Staging.  The taps of a run of pixels read, in every image it touches, one contiguous range of each
// channel plane (from the first tap of the first pixel to the last tap of the last).  That range is
// staged for a step at a time as planes of [pixel][8 channels], so that a lane's operand is one 128-bit
// read.  One staging item is 8 pixels x 8 channels: eight 16-byte loads, for NCHW an 8x8 transpose in
// registers (32 v_perm), eight 16-byte LDS writes; the filter and pixel parts share them.  Two LDS buffers
// are used in turn (one barrier per step; none at all where a wave reads only what it staged itself).
// After every eight pixels one 16-byte slot is left free: the LDS writes of neighbouring lanes, which
// are eight pixels apart, would otherwise all fall on the same banks.  A lane's nine tap addresses do
// not change from step to step and are kept in registers; a tap outside the image reads a slot of
// zeros, so the inner loop has no bounds arithmetic.
//
// Pipeline.  The loop has no branches and its waits count loads: every weight fragment is replaced, once
// used, by that of the next step, and the pixels of a step are loaded two steps ahead and go to LDS one
// step ahead.  (With a branch for partial or empty blocks in it the compiler kept two copies of these
// registers and waited for all loads at the end of every step; channels and blocks beyond the last are
// read as zeros instead, and layers with empty blocks have an instance of their own, FULL = false.)
//
// What bounds it: the vector-memory pipe, 64 bytes a cycle and compute unit.  2 x 2 blocks take 18 weight
// loads of 1 KB and 8 or more of pixels per wave for 36 matrix instructions of 32 cycles: with two such
// workgroups per compute unit a step takes 3000 cycles, of which the matrix units are busy 2300.  Around
// the loop a workgroup spends some 7000 cycles until its first operands are there and 4000 on the
// reduction and the stores, which is 40 to 60 % of the layers below.  With few workgroups that is all.
// Stride 2 stages four input pixels per output pixel, so there the filter parts matter most.
// Measured on one MI355X, the seven ResNet-50 3x3 shapes, NCHW, in us, calls back to back in a graph
// (in brackets: with three taps of weights and one step of pixels ahead, and without filter parts):
//   one image    64@56 5.3 (5.2)   128@56/2 6.9 (9.0)  128@28 5.7 (5.4)  256@28/2 9.3 (10.8)
//                256@14 6.6 (7.2)  512@14/2 9.1 (10.3)  512@7 10.1 (13.1)
//   32 images    64@56 16.4 (18.7)  128@56/2 15.4 (29.3)  128@28 14.5 (16.6)  256@28/2 16.2 (28.9)
//                256@14 14.7 (16.0)  512@14/2 18.9 (30.7)  512@7 17.6 (25.0)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <string>
#include <type_traits>

#include "pconv_fast_div.h"
#include "pconv_flat_loads.h"
#include "pconv_internal.h"

namespace pconv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct FlatArgs {
    const uint16_t *x; uint16_t *y; const float *bias;
    const uint16_t *wd;             // [fblocks][wd_row][9][32][16] bf16 bit patterns
    const uint32_t *nz;             // [cb16 / 2][fblocks]: bit (2 * tap + half)
    int c_in, w, c_out, hw, wo, howo, h;
    int stride, relu;
    int cb16, fblocks;              // blocks of 16 channels that hold any, blocks of 32 filters
    uint32_t x_bytes, wd_bytes;     // sizes of x (below 2^31) and wd
    int iters;                      // steps of a channel part
    int wd_row;                     // blocks of 16 channels in a row of wd: an even number and one of zeros
    int total;                      // output pixels of the batch
    int rhw;                        // h * w rounded up to 8
    FastDiv div_howo, div_wo, div_rhw;
    int wp_log2, wf_log2, wk;
    int bias_at;                    // where the bias lies in LDS, in floats
    int plane;                      // 16-byte slots of a staged plane
    int tiles, fgroups, filter_major;
    int inner; FastDiv div_inner;   // tiles if filter_major, fgroups otherwise
};

// 16 bytes at byte offset `lane` + `uniform` of a buffer; no more than an element's alignment is needed
__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t buf, uint32_t lane, uint32_t uniform)
{
    return __builtin_amdgcn_raw_buffer_load_b128(buf, int(lane), int(uniform), 0);
}

template <int LAYOUT, int MB, int NB, int R, int KB, int THREADS, bool FULL, bool ODD>
__global__ void __launch_bounds__(THREADS, MB * NB == 8 ? 1 : 2)
conv_flat_kernel(const FlatArgs a)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 slots[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part_log2 = a.wp_log2 + a.wf_log2;                               // waves of a channel part
    const int wpi = wave & ((1 << a.wp_log2) - 1), wfi = (wave >> a.wp_log2) & ((1 << a.wf_log2) - 1), wki = wave >> part_log2;
    const int col = lane & 31, kg = lane >> 5;

    // Workgroups whose ids are equal mod 8 run on one XCD (one L2): each gets a contiguous eighth of
    // the (tile, filter group) pairs, ordered so that neighbours share the larger of the two operands.
    const int pairs = a.tiles * a.fgroups;
    const int u = int(blockIdx.x & 7) * ((pairs + 7) >> 3) + int(blockIdx.x >> 3);
    if (u >= pairs || int(blockIdx.x >> 3) >= ((pairs + 7) >> 3)) return;
    const int outer = fast_div(u, a.div_inner), inner = u - outer * a.inner;
    const int tile = a.filter_major ? inner : outer, fg = a.filter_major ? outer : inner;

    // ---- weights: a wave's fragments of a block of channels are 9 KB in a row per block of filters ----
    // The fragments of a whole step (KB blocks of 16 channels) stay in registers; one that has been used
    // is replaced at once by that of the next step, so a load has a step's matrix instructions to arrive in.
    constexpr int Q = 9 * KB;                        // (block of channels, tap) pairs of a step
    int fb[MB];                      // (a block beyond the last one repeats it; its sums are not stored)
#pragma unroll
    for (int m = 0; m < MB; ++m) fb[m] = min(((fg << a.wf_log2) + wfi) * MB + m, a.fblocks - 1);
    u32x4 wf[Q][MB];
    const __amdgpu_buffer_rsrc_t wbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.wd), 0, a.wd_bytes, 0x00020000);
    // (ODD: the buffer begins and ends at whole dwords)
    const uint32_t x_lead = ODD ? uint32_t(reinterpret_cast<uintptr_t>(a.x)) & 2u : 0u;
    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a.x) - x_lead / 2, 0,
                                                                           ODD ? (x_lead + a.x_bytes + 3u) & ~3u : a.x_bytes, 0x00020000);
    const uint32_t wlane = uint32_t(lane & 31) * 32u + uint32_t(kg) * 16u;
    auto load_weight = [&](int g, int q, int m) {
        // (beyond the last block: the block of zeros at the end of the row)
        const int block = fb[m] * a.wd_row + min(g * KB + q / 9, a.wd_row - 1);
        wf[q][m] = load16(wbuf, wlane + uint32_t(q % 9 % 4) * 1024u, (uint32_t(block) * 9u + uint32_t(q % 9 / 4 * 4)) * 1024u);
    };

    // ---- the run of output pixels and the input ranges it reads ----
    const int p0 = tile * (NB * 32 << a.wp_log2);
    const int p_end = min(p0 + (NB * 32 << a.wp_log2), a.total);
    const int img0 = fast_div(p0, a.div_howo), img_last = fast_div(p_end - 1, a.div_howo);
    auto centre = [&](int r) { const int oy = fast_div(r, a.div_wo); return (oy * a.w + (r - oy * a.wo)) * a.stride; };
    const int lo0 = max(0, min(centre(p0 - img0 * a.howo) - a.w - 1, a.hw - 8)) & ~7;
    const int hi_last = min(a.hw, centre(p_end - 1 - img_last * a.howo) + a.w + 2);
    const int base1 = ((img_last == img0 ? hi_last : a.hw) - lo0 + 7) & ~7;      // staged position of the second image
    const int staged = img_last == img0 ? base1 : base1 + (img_last - img0 - 1) * a.rhw + ((hi_last + 7) & ~7);

    // ---- what this thread stages, the same for every step ----
    constexpr int PLANES = 2 * KB;                                             // planes of 8 channels
    const int block_slots = 2 * a.plane + 1;                                   // two planes and a slot of zeros
    const int buf_slots = a.wk * KB * block_slots;
    const int tid_g = int(threadIdx.x) & ((64 << part_log2) - 1);               // thread within the channel part
    const int g_item = tid_g & (PLANES - 1);                                   // which plane
    const uint32_t plane_step = uint32_t(a.hw) * 2u, item_step = (LAYOUT == PCONV_NCHW ? plane_step : 2u) * 8u * uint32_t(g_item);
    uint32_t src[R];                                                           // byte offset of the item's first element
    int dst[R], dst_step[R];                                                   // slot of its first pixel; pixel at which a free slot is stepped over
#pragma unroll
    for (int i = 0; i < R; ++i) {
        // A thread without an item of its own does one of the first 2^k once more: the same bytes to the
        // same place, and the loop needs no branches.
        const int own = tid_g / PLANES + i * ((64 / PLANES) << part_log2);
        const int pos = (own * 8 < staged ? own : own & ((1 << (31 - __builtin_clz(uint32_t(staged) >> 3))) - 1)) * 8;
        int img = img0, q = lo0 + pos;
        if (pos >= base1) {
            const int t = pos - base1, s = fast_div(t, a.div_rhw);
            img = img0 + 1 + s; q = t - s * a.rhw;
        }
        // the last item of a plane is moved back to end with it (and writes some pixels a second time)
        const int q8 = min(q, a.hw - 8), wpos = pos - (q - q8);
        const uint32_t e = LAYOUT == PCONV_NCHW ? uint32_t(img * a.c_in * a.hw + q8)
                                                : uint32_t((img * a.hw + q8) * a.c_in);
        src[i] = e * 2u + item_step + x_lead;
        dst[i] = (wki * KB + (g_item >> 1)) * block_slots + (g_item & 1) * a.plane + wpos + (wpos >> 3);
        dst_step[i] = 8 - (wpos & 7);
    }
    // Pixels on their way to LDS.  ODD: where the planes of channels have an odd number of pixels, half of the
    // items are not aligned to dwords, and such a load costs four times an aligned one: the dwords around an
    // item are loaded instead, the fifth, if there is one, into `fifth` (512@7: 11.4 -> 10.1 us with one
    // image, 18.6 -> 17.6 with 32).
    u32x4 raw[R][8];
    uint32_t fifth[R][8];
    // (a channel beyond c_in is read as zeros: see flat_load)
    auto load_rows = [&](int g, u32x4 (&raw)[R][8], uint32_t (&fifth)[R][8], int j0, int j1) {          // channels (NHWC: pixels) j0 ... j1 - 1 of the items
        const int c0 = g * (16 * KB);
#pragma unroll
        for (int j = j0; j < j1; ++j) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const FlatLoad at = flat_load<LAYOUT == PCONV_NCHW, ODD>(src[i], g_item, j, c0, a.c_in, plane_step);
                raw[i][j] = load16(xbuf, at.lane, at.uniform);
                if (ODD) {
                    const FlatLoad behind = flat_load_fifth(at, src[i], j);
                    fifth[i][j] = __builtin_amdgcn_raw_buffer_load_b32(xbuf, int(behind.lane), int(behind.uniform), 0);
                }
            }
        }
    };
    // ODD: eight pixels out of the five dwords around them
    auto align_rows = [&](u32x4 (&raw)[R][8], const uint32_t (&fifth)[R][8]) {
        if (!ODD) return;
#pragma unroll
        for (int i = 0; i < R; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t shift = ((src[i] + 2u * (j & 1)) & 2u) * 8u;
                const u32x4 d = raw[i][j];
                raw[i][j] = u32x4{__builtin_amdgcn_alignbit(d[1], d[0], shift), __builtin_amdgcn_alignbit(d[2], d[1], shift),
                                  __builtin_amdgcn_alignbit(d[3], d[2], shift), __builtin_amdgcn_alignbit(fifth[i][j], d[3], shift)};
            }
    };
    // pixel j of this thread's items to LDS
    auto store_pixel = [&](int buf, int j, const u32x4 (&raw)[R][8]) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            u32x4 *lp = slots + buf * buf_slots + dst[i];
            u32x4 *lp1 = lp + 1;
            u32x4 v;
            if (LAYOUT == PCONV_NCHW) {
                // 16-bit half j % 2 of dword j / 2 of the eight channel rows
                const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
                for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_perm(raw[i][2 * k + 1][j >> 1], raw[i][2 * k][j >> 1], sel);
            } else {
                v = raw[i][j];
            }
            (j >= dst_step[i] ? lp1 : lp)[j] = v;
        }
    };
    // The prologue asks for everything that the first step needs, and the pixels of the second, in the
    // order of the loop below (the waits in the loop count what was asked for since); the tap addresses
    // are worked out in between, while the memory pipe is busy.
    constexpr int TURN = Q / 3;                      // the tap of a step at which the next step's pixels go to LDS
    u32x4 raw0[R][8];
    uint32_t fifth0[R][8];
    load_rows(wki, raw0, fifth0, 0, 8);
    __builtin_amdgcn_sched_barrier(0);

    // ---- this lane's tap addresses (bytes, in buffer 0) ----
    int addr[9][NB];
    const int part_at = wki * KB * block_slots * 16, zeros_at = part_at + 2 * a.plane * 16;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int p = p0 + (wpi * NB + j) * 32 + col, pc = min(p, a.total - 1);
        const int img = fast_div(pc, a.div_howo), r = pc - img * a.howo;
        const int oy = fast_div(r, a.div_wo), ox = r - oy * a.wo;
        const int iy = oy * a.stride, ix = ox * a.stride;
        const int pos = (img == img0 ? -lo0 : base1 + (img - img0 - 1) * a.rhw) + iy * a.w + ix;
        const int lane_at = part_at + kg * a.plane * 16;
        // (no short-circuits: selects, not branches)
        const int col_ok[3] = {ix > 0, 1, ix + 1 < a.w};
        const int row_ok[3] = {(p < p_end) & (iy > 0), p < p_end, (p < p_end) & (iy + 1 < a.h)};
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            const int t = pos + (q / 3 - 1) * a.w + (q % 3 - 1);
            addr[q][j] = row_ok[q / 3] & col_ok[q % 3] ? lane_at + ((t + (t >> 3)) << 4) : zeros_at;
        }
        // (half of the weights after the first pixel block's addresses, half after the last one's)
        if (j == 0) {
#pragma unroll
            for (int q = 0; q < TURN; ++q)
#pragma unroll
                for (int m = 0; m < MB; ++m) load_weight(wki, q, m);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    load_rows(a.wk + wki, raw, fifth, 0, 8);     // (also where there is no second step: it reads nothing)
#pragma unroll
    for (int q = TURN; q < Q; ++q)
#pragma unroll
        for (int m = 0; m < MB; ++m) load_weight(wki, q, m);

    f32x16 acc[MB][NB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[m][j] = 0.0f;

    // bias of the workgroup's filters, behind everything else in LDS (-0 where there is none: x + -0 = x)
    float *bias_lds = reinterpret_cast<float *>(slots) + a.bias_at;
    if (int(threadIdx.x) < MB * 32 << a.wf_log2) {
        const int f = (fg << a.wf_log2) * MB * 32 + int(threadIdx.x);
        bias_lds[threadIdx.x] = a.bias && f < a.c_out ? a.bias[f] : -0.0f;
    }
    if (int(threadIdx.x) < 2 * a.wk * KB) slots[threadIdx.x * block_slots + 2 * a.plane] = u32x4{0u, 0u, 0u, 0u};
    align_rows(raw0, fifth0);
#pragma unroll
    for (int j = 0; j < 8; ++j) store_pixel(0, j, raw0);
    const int iters = a.iters;
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

    // One step: KB blocks of channels.  Half way the pixels of the next step, whose loads have had a
    // step to arrive, go to the other LDS buffer, and the loads of the step after that are issued (which
    // read nothing beyond the last channel).  AFTER: another step follows.
    auto step = [&](int it, auto after_c) {
        constexpr bool AFTER = decltype(after_c)::value;
        const int g = it * a.wk + wki, buf = it & 1;
        const char *bp = lds_bytes + buf * buf_slots * 16;
        auto fragment = [&](int q, int j) { return *reinterpret_cast<const bf16x8 *>(bp + (q / 9) * block_slots * 16 + addr[q % 9][j]); };
        uint32_t bits[KB][MB];
        if (!FULL) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int cb = g * KB + kb;
                    bits[kb][m] = cb < a.cb16 ? nz[(cb >> 1) * a.fblocks + fb[m]] >> (cb & 1) : 0u;
                }
        }
        // taps by which the pixel fragments are read ahead (the latency of LDS; registers permitting)
        constexpr int AHEAD = MB * NB == 1 ? 4 : MB * NB == 2 ? 3 : MB * NB == 4 ? 2 : 1;
        bf16x8 xv[AHEAD + 1][NB];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q)
#pragma unroll
            for (int j = 0; j < NB; ++j) xv[q][j] = fragment(q, j);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            if (q + AHEAD < Q) {
#pragma unroll
                for (int j = 0; j < NB; ++j) xv[(q + AHEAD) % (AHEAD + 1)][j] = fragment(q + AHEAD, j);
            }
            if (AFTER && q == TURN) align_rows(raw, fifth);
#pragma unroll
            for (int m = 0; m < MB; ++m)
                if (FULL || ((bits[q / 9][m] >> (2 * (q % 9))) & 1u)) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        acc[m][j] = mfma(wf[q][m], xv[q % (AHEAD + 1)][j], acc[m][j]);
                        if (FULL && AFTER && q == TURN) {
                            // (a few pixels after each matrix instruction, which keeps its unit busy meanwhile)
#pragma unroll
                            for (int k = 0; k < 8; ++k)
                                if (k * MB * NB / 8 == m * NB + j) store_pixel(buf ^ 1, k, raw);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            if (!FULL && AFTER && q == TURN) {
#pragma unroll
                for (int k = 0; k < 8; ++k) store_pixel(buf ^ 1, k, raw);
            }
            if (AFTER) {
                // (spread over the rest of the step: a load waits for the memory pipe, and the next matrix
                // instruction behind it)
                if (q >= TURN) load_rows(g + 2 * a.wk, raw, fifth, (q - TURN) * 8 / (Q - TURN), (q - TURN + 1) * 8 / (Q - TURN));
#pragma unroll
                for (int m = 0; m < MB; ++m) load_weight(g + a.wk, q, m);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (AFTER) {
            if (part_log2) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
        }
    };
#pragma unroll 1
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
    auto finish = [&](auto wk_c) {
        constexpr int WK = decltype(wk_c)::value, ROUNDS = (MB * NB * 2 + WK - 1) / WK, STEP = 64 / OCT;
        if (wki >= MB * NB * 2) return;
        const int o = lane & (OCT - 1);                                        // this lane's octet in the row, in every round
        const f32x4 *rp0 = red + (((wfi << a.wp_log2) + wpi) * G + (o & 3)) * kGroupPitch;
        auto sums = [&](int m, int j, int c, f32x4 &v0, f32x4 &v1) {
            const f32x4 *rp = rp0 + ((m * NB + j) * 4) * kGroupPitch + c;
            v0 = rp[0]; v1 = rp[32];
#pragma unroll
            for (int k = 1; k < WK; ++k) {
                rp += (G * kGroupPitch) << part_log2;
                v0 += rp[0]; v1 += rp[32];
            }
        };
        union Octet { __bf16 e[8]; uint16_t u[8]; u32x4 d; };
        auto round8 = [&](const f32x4 &v0, const f32x4 &v1, auto &&bias_of) {
            Octet out;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const float t = (k < 4 ? v0[k & 3] : v1[k & 3]) + bias_of(k);
                out.e[k] = __bf16(a.relu ? fmaxf(t, 0.0f) : t);
            }
            return out;
        };
        if (LAYOUT == PCONV_NCHW) {
            // a lane's eight pixels are the same in every round, the filters go on
            const int p = p0 + wpi * NB * 32 + 8 * o;
            const int img = fast_div(p, a.div_howo), r = p - img * a.howo;
            const bool whole = (r + 8 <= a.howo) & (p + 8 <= p_end);
            uint32_t at[8];                                                    // of each pixel in filter 0 (where they are not in a row)
            at[0] = uint32_t(img * a.c_out) * uint32_t(a.howo) + uint32_t(r);
            if (!whole) {
#pragma unroll
                for (int k = 1; k < 8; ++k) {
                    const int im = fast_div(p + k, a.div_howo);
                    at[k] = uint32_t(im * a.c_out) * uint32_t(a.howo) + uint32_t(p + k - im * a.howo);
                }
            }
            const int pixels = min(8, p_end - p);
#pragma unroll 4
            for (int i = 0; i < ROUNDS; ++i) {
                const int fl = lane / OCT + (wki + i * WK) * STEP, m = fl >> 5, c = fl & 31;
                f32x4 v0, v1;
                sums(m, o >> 2, c, v0, v1);
                const float b = bias_lds[wfi * MB * 32 + fl];
                const Octet out = round8(v0, v1, [&](int) { return b; });
                const int f = ((fg << a.wf_log2) + wfi) * MB * 32 + fl;
                if (f >= a.c_out) continue;
                uint16_t *yp = a.y + uint32_t(f) * uint32_t(a.howo);
                if (whole) {
                    __builtin_memcpy(yp + at[0], &out.d, 16);
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        if (k < pixels) yp[at[k]] = out.u[k];
                }
            }
        } else {
            // a lane's eight filters are the same in every round, the pixels go on
            const int fl = 8 * o, f = ((fg << a.wf_log2) + wfi) * MB * 32 + fl;
            float b[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) b[k] = bias_lds[wfi * MB * 32 + fl + k];
#pragma unroll 4
            for (int i = 0; i < ROUNDS; ++i) {
                const int pl = lane / OCT + (wki + i * WK) * STEP, j = pl >> 5, c = pl & 31;
                f32x4 v0, v1;
                sums(o >> 2, j, c, v0, v1);
                const Octet out = round8(v0, v1, [&](int k) { return b[k]; });
                const int p = p0 + wpi * NB * 32 + pl;
                if ((p >= p_end) | (f >= a.c_out)) continue;
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
    };
    if (a.wk == 1) finish(std::integral_constant<int, 1>{});
    else if (a.wk == 2) finish(std::integral_constant<int, 2>{});
    else if (a.wk == 4) finish(std::integral_constant<int, 4>{});
    else finish(std::integral_constant<int, 8>{});
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

template <int LAYOUT, int MB, int NB, int R, int KB, int THREADS, bool FULL, bool ODD>
hipError_t launch_flat(const FlatArgs &a, dim3 grid, dim3 block, int64_t lds, hipStream_t st, int dev)
{
    // More dynamic LDS than the default limit: raised once per device (the flag is set to the same
    // value by every thread that gets here first).
    static std::atomic<bool> attr_done[64];
    if (dev < 0 || dev >= 64 || !attr_done[dev].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_flat_kernel<LAYOUT, MB, NB, R, KB, THREADS, FULL, ODD>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsOfUnit));
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_done[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((conv_flat_kernel<LAYOUT, MB, NB, R, KB, THREADS, FULL, ODD>), grid, block, size_t(lds), st, a);
    return hipGetLastError();
}

// Launch shape: MB x NB blocks of 32 filters x 32 pixels per wave, WP pixel parts x WK channel parts x WF
// filter parts, KB blocks of 16 channels per step; R staging items per thread.
struct FlatShape { int index, mb, nb, wp, wk, kb, wf, r; int64_t plane, lds; };

// The 24 of 53 shapes measured (the four parts and both block counts in all combinations that looked
// useful) whose best is within 1 % of the best of all, on average over 192 layers: see choose_flat.
constexpr int kShapes[][6] = {
    {2, 2, 1, 4, 1, 1}, {1, 2, 4, 1, 1, 1}, {1, 2, 2, 2, 1, 1}, {1, 2, 1, 4, 1, 1}, {1, 2, 1, 4, 2, 1}, {1, 1, 2, 2, 2, 1},
    {1, 2, 4, 1, 2, 1}, {1, 1, 2, 2, 1, 1}, {1, 1, 1, 8, 1, 1}, {1, 4, 4, 1, 1, 1}, {1, 4, 2, 2, 1, 1}, {1, 2, 2, 1, 1, 2},
    {1, 2, 1, 2, 1, 2}, {1, 1, 1, 8, 2, 1}, {2, 2, 4, 1, 1, 2}, {1, 1, 1, 4, 1, 2}, {1, 1, 4, 1, 1, 2}, {2, 4, 2, 1, 1, 2},
    {1, 1, 1, 1, 2, 4}, {2, 2, 2, 2, 1, 2}, {2, 2, 1, 2, 1, 2}, {1, 2, 1, 4, 1, 2}, {2, 2, 2, 1, 1, 2}, {1, 2, 4, 1, 1, 2},
    {1, 1, 4, 1, 1, 1}};            // (the last for layers of one block each way)
constexpr int kNumShapes = int(sizeof kShapes / sizeof kShapes[0]);
std::atomic<int> g_force_shape{-1};      // test override, see set_flat_shape

// Combinations whose working set outgrows the registers of a wave are not built.
constexpr bool fits_registers(int mb, int nb, int kb, int r, bool odd)
{
    if (r == 1) return true;
    return mb * nb == 8 ? !odd : nb < 4 && mb == 1 && !(odd && kb == 2);
}

// The shape with the smallest estimate of the layer's time, in microseconds; false if the kernel does
// not serve the call.  Few workgroups: the time of one, that is its start, in which all its waves send for
// their weights and pixels through one memory pipe, and its steps.  Many: what a compute unit spends on a
// workgroup, per wave and block of outputs, per wave and step for every load and every LDS access.  The
// constants are a fit to these shapes on 150 layers drawn at random (16 to 512 channels, 7 to 224 pixels
// square and not, both strides and layouts, 1 to 64 images) and the seven 3x3 shapes of ResNet-50 with 1,
// 8 and 32 images: the shape chosen takes 2.6 % longer than the fastest one on average, 30 % at most
// (352->448@40/2, 22 images).
bool choose_flat(const pconv_handle *h, int n, int hin, int win, int stride, int layout, FlatShape &best)
{
    const int hw = hin * win, wo = (win - 1) / stride + 1, howo = ((hin - 1) / stride + 1) * wo, total = n * howo;
    const int cb16 = (h->c_in + 15) / 16, wd_row = (h->c_in + 31) / 32 * 2 + 1, fblocks = (h->c_out + 31) / 32;
    // (a staging item is eight pixels of a plane; NHWC pixels are read in whole octets of channels)
    if (hw < 8 || (layout == PCONV_NHWC && h->c_in % 8 != 0)) return false;
    if (int64_t(fblocks) * wd_row * 9 * 1024 >= (int64_t(1) << 32)) return false;   // (32-bit weight offsets)
    best = FlatShape{};
    double best_time = 0.0;
    const int cus = h->cus > 0 ? h->cus : 256, forced = g_force_shape.load();
    int64_t bounds[5] = {0, 0, 0, 0, 0};                                        // of runs of 32, 64, 128, 256 and 512 pixels, once asked for
    for (int k = 0; k < kNumShapes; ++k) {
        const auto &c = kShapes[k];
        FlatShape s{k, c[0], c[1], c[2], c[3], c[4], c[5], 1, 0, 0};
        if (forced >= 0 && k != forced) continue;
        if (s.mb * s.wf > fblocks + s.mb - 1 || s.mb > fblocks || s.wk > (cb16 + s.kb - 1) / s.kb || s.kb > cb16) continue;
        const int np = 32 * s.nb * s.wp, part = s.wp * s.wf, waves = part * s.wk;
        int64_t &bound = bounds[31 - __builtin_clz(unsigned(np)) - 5];
        if (bound == 0) bound = staged_bound(np, hw, howo, win, wo, stride);
        s.plane = bound + bound / 8;
        s.lds = std::max<int64_t>(2 * s.wk * s.kb * (2 * s.plane + 1) * 16, int64_t(waves) * s.mb * s.nb * 4 * 65 * 16) + 128 * int64_t(s.mb * s.wf);
        const int64_t items = bound / 4 * s.kb;
        s.r = items <= 64 * part ? 1 : 2;
        if (!fits_registers(s.mb, s.nb, s.kb, s.r, layout == PCONV_NCHW && hw % 2 != 0)) continue;
        if (items > 64 * part * s.r || s.lds > kLdsOfUnit) continue;
        const int iters = ((cb16 + s.kb - 1) / s.kb + s.wk - 1) / s.wk;
        const int64_t tiles = (total + np - 1) / np, fgroups = (fblocks + s.mb * s.wf - 1) / (s.mb * s.wf);
        const double groups = double(tiles) * fgroups / cus;
        const int resident = int(std::max<int64_t>(1, std::min<int64_t>(kLdsOfUnit / s.lds, (s.mb * s.nb < 8 ? 8 : 4) / waves)));
        const bool odd = layout == PCONV_NCHW && hw % 2 != 0;
        const int staging = 8 * s.r, loads = 9 * s.kb * s.mb + staging * (odd ? 2 : 1), lds_ops = 9 * s.kb * s.nb + staging;
        const double chain = 2.4 + 0.0052 * waves * loads + iters * (0.054 + 0.0178 * 9 * s.kb * s.mb * s.nb + 0.0051 * waves * loads);
        const double busy = waves * (0.025 * s.mb * s.nb + 0.0062 * (iters + 1) * loads + 0.0057 * iters * lds_ops);
        const double rounds = std::ceil(groups / resident);
        const double lo = std::min(groups * busy, rounds * chain), hi = std::max(groups * busy, rounds * chain);
        const double time = hi + 0.3 * lo;
        if (best.mb == 0 || time < best_time) { best = s; best_time = time; }
    }
    if (best.mb == 0) return false;
    const int np = 32 * best.nb * best.wp;
    return int64_t((total + np - 1) / np) * fblocks <= 0x3FFFFFFF;
}

}  // namespace

void set_flat_shape(int index) { g_force_shape.store(index >= 0 && index < kNumShapes ? index : -1); }

int flat_shape_of(const pconv_handle *h, int n, int hin, int win, int stride, int layout)
{
    FlatShape s;
    return choose_flat(h, n, hin, win, stride, layout, s) ? s.index : -1;
}

// choose_flat, or what it chose for the same call before
static bool flat_shape(const pconv_handle *h, int n, int hin, int win, int stride, int layout, FlatShape &s)
{
    if (g_force_shape.load() >= 0) return choose_flat(h, n, hin, win, stride, layout, s);
    {
        const std::lock_guard<std::mutex> lock(h->flat_mutex);
        for (const FlatCall &c : h->flat_calls)
            if (c.n == n && c.h == hin && c.w == win && c.stride == stride && c.layout == layout) {
                const auto &k = kShapes[c.index];
                s = FlatShape{c.index, k[0], k[1], k[2], k[3], k[4], k[5], c.r, c.plane, c.lds};
                return true;
            }
    }
    if (!choose_flat(h, n, hin, win, stride, layout, s)) return false;
    if (g_force_shape.load() >= 0) return true;                                // (pinned meanwhile: not the call's own shape)
    const std::lock_guard<std::mutex> lock(h->flat_mutex);
    h->flat_calls[h->flat_next++ % 4] = FlatCall{n, hin, win, stride, layout, s.index, s.r, s.plane, s.lds};
    return true;
}

bool launch_conv_flat(const pconv_handle *h, const void *x, void *y, const float *bias, int n, int hin, int win,
                      int stride, int layout, int relu, void *stream, int &rc)
{
    FlatShape best;
    if (!flat_shape(h, n, hin, win, stride, layout, best)) return false;
    FlatArgs a;
    a.x = static_cast<const uint16_t *>(x); a.y = static_cast<uint16_t *>(y); a.bias = bias;
    a.wd = h->d_wdense; a.nz = h->d_wnz;
    a.c_in = h->c_in; a.h = hin; a.w = win; a.c_out = h->c_out;
    a.x_bytes = uint32_t(int64_t(n) * h->c_in * hin * win * 2);
    a.wd_bytes = uint32_t(int64_t((h->c_out + 31) / 32) * ((h->c_in + 31) / 32 * 2 + 1) * 9 * 1024);
    const int ho = (hin - 1) / stride + 1;
    a.wo = (win - 1) / stride + 1; a.hw = hin * win; a.howo = ho * a.wo;
    a.stride = stride; a.relu = relu;
    a.cb16 = (h->c_in + 15) / 16; a.wd_row = (h->c_in + 31) / 32 * 2 + 1; a.fblocks = (h->c_out + 31) / 32;
    a.total = n * a.howo;
    a.rhw = (a.hw + 7) & ~7;
    a.div_howo = make_fast_div(uint32_t(a.howo)); a.div_wo = make_fast_div(uint32_t(a.wo));
    a.div_rhw = make_fast_div(uint32_t(a.rhw));
    const int mb = best.mb, nb = best.nb, wp = best.wp, wk = best.wk, wf = best.wf;
    a.iters = ((a.cb16 + best.kb - 1) / best.kb + wk - 1) / wk;
    const int np = 32 * nb * wp;
    const int64_t lds = best.lds, plane = best.plane;
    a.bias_at = int(lds / 4) - 32 * mb * wf;
    a.wp_log2 = wp == 4 ? 2 : wp == 2 ? 1 : 0; a.wf_log2 = wf == 8 ? 3 : wf == 4 ? 2 : wf == 2 ? 1 : 0; a.wk = wk; a.plane = int(plane);
    a.tiles = (a.total + np - 1) / np; a.fgroups = (a.fblocks + mb * wf - 1) / (mb * wf);
    a.filter_major = int64_t(h->c_out) * 9 > int64_t(n) * a.hw;
    a.inner = a.filter_major ? a.tiles : a.fgroups; a.div_inner = make_fast_div(uint32_t(a.inner));
    const int64_t pairs = int64_t(a.tiles) * a.fgroups;
    const dim3 grid{unsigned((pairs + 7) / 8 * 8)}, block{unsigned(64 * wp * wf * wk)};
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipErrorInvalidValue;
    auto pick = [&](auto lay, auto rr, auto mm, auto nn, auto kk) {
        constexpr int L = decltype(lay)::value, RR = decltype(rr)::value, M = decltype(mm)::value, N = decltype(nn)::value,
                      K = decltype(kk)::value;
        if (mb != M || nb != N || best.kb != K) return;
        constexpr int most = M * N < 8 ? 512 : 256;
        if (int(block.x) > most) return;
        constexpr bool nchw = L == PCONV_NCHW;
        if constexpr (nchw && fits_registers(M, N, K, RR, true)) {
            if (a.hw % 2 != 0) {
                if (h->wd_full) e = launch_flat<L, M, N, RR, K, most, true, true>(a, grid, block, lds, st, h->device);
                else e = launch_flat<L, M, N, RR, K, most, false, true>(a, grid, block, lds, st, h->device);
                return;
            }
        }
        if constexpr (fits_registers(M, N, K, RR, false)) {
            if (h->wd_full) e = launch_flat<L, M, N, RR, K, most, true, false>(a, grid, block, lds, st, h->device);
            else e = launch_flat<L, M, N, RR, K, most, false, false>(a, grid, block, lds, st, h->device);
        }
    };
    using std::integral_constant;
    auto pick_shape = [&](auto lay, auto rr) {
        const integral_constant<int, 1> one; const integral_constant<int, 2> two; const integral_constant<int, 4> four;
        pick(lay, rr, two, two, one);
        pick(lay, rr, two, four, one);
        pick(lay, rr, one, four, one);
        pick(lay, rr, one, two, one);
        pick(lay, rr, one, two, two);
        pick(lay, rr, one, one, one);
        pick(lay, rr, one, one, two);
    };
    const integral_constant<int, PCONV_NCHW> nchw; const integral_constant<int, PCONV_NHWC> nhwc;
    if (layout == PCONV_NHWC) {
        if (best.r == 1) pick_shape(nhwc, integral_constant<int, 1>{});
        else pick_shape(nhwc, integral_constant<int, 2>{});
    } else {
        if (best.r == 1) pick_shape(nchw, integral_constant<int, 1>{});
        else pick_shape(nchw, integral_constant<int, 2>{});
    }
    rc = PCONV_OK;
    if (e != hipSuccess) {
        set_error(std::string("pconv_conv2d (matrix-core kernel): ") + hipGetErrorName(e));
        rc = PCONV_HIP_ERROR;
    }
    return true;
}

}  // namespace pconv
