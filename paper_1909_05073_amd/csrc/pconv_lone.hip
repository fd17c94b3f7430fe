// fp32 PCONV for layers with few to middling numbers of units of work: every wave on its own (NCHW, stride 1 and 2).
//
// A workgroup is one tile of up to 64 patches (4x4 output pixels, one per lane) and one block of four
// filters, or two of its four slots (halves, where there are too few blocks for the chip).  Its waves, 16, 8 or 4
// (one, two or four workgroups to a compute unit), share out the visits of those filters: the channels that have a
// record, in an order fixed at pack time.  A wave loads the six input rows of a channel straight into the registers of the record
// loop, takes the columns beside the patch out of the neighbouring lanes, runs the records and goes on:
// nothing is staged and there is nothing to wait for but its own loads.  The visit after next is read from
// the list and the first record words are on their way while the rows are.  At the end the partial
// sums are added through LDS.
//
// What bounds it: the vector-memory pipe, and the issue of vector instructions behind it.  A visit takes 1360 cycles of a wave
// in the oldest four of 16 waves and 1910 in the youngest (hence portions by age, see the packer), so a compute unit ends
// one in 100 cycles, and its six 1 KB loads take the pipe 16.5 cycles each; its 97 FMAs (1.5 records) of 2.4 cycles and 12 moves
// between lanes are 260 of the 400 cycles that a SIMD has for it.  Over the whole kernel (256 channels @56, counters) the pipe has
// 18 700 of the 35 000 cycles that a wave lives and vector issue 16 500; with 4 waves and few records a visit (512 @28, 64 images,
// uneven) 62 and 38 %, stride 2 62 and 23.  Fewer loads by themselves do not help: the rows staged in LDS as one run of memory,
// one to five loads for six, the next channel's under the records: 19.8 us for 18.1 on the first layer, 512 @14, 32 images, 4 waves
// 104 for 92.  Start 3600 cycles, sums and stores 5000 with 16 waves.  One image, us: 256 channels @56 16.4, 512 @14 18.6, 512 @28 22,
// 16 @16 5.7 for the kernel.
//
// Waves of a workgroup.  With 16 the end of every workgroup, its start and a last round of few workgroups leave the
// compute unit to itself; with 8 or 4 other workgroups run meanwhile and a round is half or a quarter as long, but too few
// workgroups leave it with few waves.  us with 16, 8 and 4 (see the estimates in pconv_tiled.hip): 64 channels @224, one
// image 33, 23, 19; 128 @112 23, 19, 22; 256 @56 18, 22, 33; 512 @14, 32 images 113, 105, 100; 256 @28, 32 images 118, 99, 93.
//
// Tiles.  Where it costs little, a tile is a whole number of patch rows, so that every column beside a
// patch is in the next lane or outside the image.  Otherwise (CUT: rows of more than 64 patches, or tiles that
// would leave many lanes empty) the first and the last lane's outer columns are loaded apart, twelve words.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <type_traits>

#include "pconv_fast_div.h"
#include "pconv_internal.h"
#include "pconv_tiled_codes.h"

namespace pconv {

namespace {

constexpr int FB = kTileFB;
constexpr uint32_t kOutOfRange = 0x80000000u;      // byte offset beyond any tensor served here
constexpr int kBatch = 64;                         // records at hand per wave: one per lane

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct LoneArgs {
    const float *x; float *y; const float *bias;
    const int32_t *slot_filter; const uint32_t *bounds, *visits, *meta; const float4 *w4;
    int c_in, h, w, c_out;
    int px, per_img, n_patches, patch_base, lanes; // patches of a row, of an image, of the batch, before the first tile, of a tile
    int n_units, n_groups, halves;
    int relu, pool, sub2;
    uint32_t n_records, x_bytes;
    FastDiv div_img, div_px, div_groups;
};

// OVER: columns by which the last patch of a row is shifted left.  CUT: tiles may begin and end inside a row.  LAST:
// outputs with channels last.  NW: waves.  SUB2: stride 2 with all patches starting at even columns (an even width): only
// the outputs that are stored are formed, a quarter of the FMAs, out of the first five rows and the column to the left.
template <int OVER, bool CUT, bool LAST, int NW, bool SUB2>
__global__ void __launch_bounds__(NW * 64, 4)      // 4 waves per SIMD: at most 128 VGPRs
conv_lone_kernel(const LoneArgs a)
{
    extern __shared__ __attribute__((aligned(16))) v4f lds4[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    auto fresh_lane = [&]() { int l = threadIdx.x & 63; asm volatile("" : "+v"(l)); return l; };
    // (XCD s, the workgroups whose ids are s mod 8, gets the s-th eighth of the units, so that its L2 serves few tiles)
    const int per_xcd = (a.n_units + 7) >> 3;
    const int unit = int(blockIdx.x & 7) * per_xcd + int(blockIdx.x >> 3);
    if (unit >= a.n_units || int(blockIdx.x >> 3) >= per_xcd) return;
    const int tile = fast_div(unit, a.div_groups), group = unit - tile * a.n_groups;
    const int half = a.halves ? group & 1 : -1;    // slots 0 and 1, or 2 and 3; -1: all
    const int fblk = a.halves ? group >> 1 : group;

    // ---- this wave's channels ----
    // A visit is a channel with a record of the workgroup's filters: its first record, its channel and (from
    // bit 16 on) the number of records.  The workgroups of a tile walk the same channels; each starts a
    // little further on, so that what it asks for was fetched into the L2 by its neighbour shortly before.
    // Where a wave starts follows from the filters alone, never from the tile: two tiles that both
    // store the columns an overlapping last patch shares must have added them in one order.
    // (constant address space: scalar loads)
    typedef const uint32_t __attribute__((address_space(4))) *ConstWords;
    auto constant = [](const void *p) { return reinterpret_cast<ConstWords>(reinterpret_cast<uintptr_t>(p)); };
    // (the portions are for 16 waves; with fewer, each gets the same number of visits)
    const ConstWords bounds = constant(a.bounds) + (fblk * 3 + half + 1) * (kLoneWaves + 1);
    const int v_first = int(bounds[0]), v_all = int(bounds[kLoneWaves]) - v_first;
    const int v_lo = NW == kLoneWaves ? int(bounds[wave]) : v_first + v_all * wave / NW;
    const int v_hi = NW == kLoneWaves ? int(bounds[wave + 1]) : v_first + v_all * (wave + 1) / NW, n_visits = v_hi - v_lo;
    // (waves from `parts` on have no visits; an earlier one may have none either, beside a very costly visit: it adds zeros)
    const int parts = NW == kLoneWaves ? max(1, min(NW, v_all)) : NW;
    struct Visit { uint32_t record, channel_count; };
    const ConstWords visits = constant(a.visits), meta = constant(a.meta);
    auto visit_at = [&](int v) { return Visit{visits[2 * v], visits[2 * v + 1]}; };
    auto after = [&](int v) { return v + 1 < v_hi ? v + 1 : v_lo; };
    int v = v_lo + ((group & 15) * n_visits >> 4);
    // (a wave without visits reads the padding at the end of the list)
    Visit now = visit_at(v), next = visit_at(after(v));
    const uint32_t k_lo = visits[2 * v_lo];
    // what the end needs: filter and bias of the slots that this wave adds up: one in each pass, both with four waves
    // (SUB2: one, all in one pass)
    constexpr int SLOTS = SUB2 ? 1 : NW < 8 ? FB : FB / 2, PER_PASS = 2 * SLOTS / FB;
    const int u = NW < 8 ? 0 : (wave >> 2) & 1, i = wave & 3;
    int filter[SLOTS];
    float slot_bias[SLOTS];
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
        filter[k] = int(constant(a.slot_filter)[fblk * FB + (SUB2 ? wave & (FB - 1) : NW < 8 ? k : 2 * k + u)]);
        slot_bias[k] = a.bias && filter[k] >= 0 ? __uint_as_float(constant(a.bias)[filter[k]]) : 0.0f;
    }

    // ---- this lane's patch ----
    // (worked out again at the end: few vector registers may stay live across the record loop)
    struct Patch { bool valid; int n, y0, x0, col; };
    auto patch_of = [&](int ln) {
        // (the last patch of a row is shifted left so that it ends at the image edge)
        const int pidx = a.patch_base + tile * a.lanes + ln;
        Patch p;
        p.valid = ln < a.lanes && pidx < a.n_patches;
        p.n = p.valid ? fast_div(pidx, a.div_img) : 0;
        const int prem = p.valid ? pidx - p.n * a.per_img : 0, prow = fast_div(prem, a.div_px);
        p.col = prem - prow * a.px;
        p.y0 = prow * 4; p.x0 = min(p.col * 4, a.w - 4);
        return p;
    };
    // byte offset in channel 0 of the six rows, beyond the tensor where the row is outside the image
    uint32_t row_at[6];
    // what the columns beside the patch are: bit 0, 1: the left, right one lies in the image; beside the last
    // patch of a row, which is shifted, the next column is another one of the neighbour's: bit 2: this
    // patch gives column 3 - over to the right instead of 3; bit 3: it gives `over` to the left instead of 0;
    // bits 4, 5: the first, the last lane
    int beside;
    {
        const Patch p = patch_of(lane);
        const int at0 = (p.n * a.c_in * a.h + (p.y0 - 1)) * a.w + p.x0;
#pragma unroll
        for (int r = 0; r < 6; ++r)
            row_at[r] = p.valid && uint32_t(p.y0 - 1 + r) < uint32_t(a.h) ? uint32_t(at0 + r * a.w) * 4u : kOutOfRange;
        beside = (p.col > 0) | (p.col < a.px - 1) << 1 | (p.col == a.px - 2) << 2 | (p.col == a.px - 1) << 3 | (lane == 0) << 4 | (lane == 63) << 5;
    }
    auto mask = [&](int bit) { return uint32_t(beside << (31 - bit) >> 31); };  // all ones where the bit is set

    const __amdgpu_buffer_rsrc_t xbuf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x), 0, a.x_bytes, 0x00020000);
    const uint32_t plane = uint32_t(a.h) * uint32_t(a.w) * 4u;
    v4f rows[6];
    // CUT: word 2 r is left of lane 0's patch in row r, word 2 r + 1 right of lane 63's
    uint32_t outer_at = kOutOfRange;
    float outer = 0.0f;
    if (CUT) {
        const Patch p = patch_of(lane & 1 ? 63 : 0);
        const int r = lane >> 1, iy = p.y0 - 1 + r, ix = lane & 1 ? p.x0 + 4 : p.x0 - 1;
        if (lane < 12 && p.valid && uint32_t(iy) < uint32_t(a.h) && uint32_t(ix) < uint32_t(a.w))
            outer_at = uint32_t((p.n * a.c_in * a.h + iy) * a.w + ix) * 4u;
    }
    auto load_rows = [&](int c) {
        const int at = __builtin_amdgcn_readfirstlane(int(uint32_t(c) * plane));
#pragma unroll
        for (int r = 0; r < (SUB2 ? 5 : 6); ++r) rows[r] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(xbuf, int(row_at[r]), at, 0));
        if (CUT) outer = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xbuf, int(outer_at), at, 0));
    };
    if (n_visits > 0) load_rows(int(now.channel_count & 0xFFFFu));

    v16f acc[FB];
    float zero = 0.0f;
    asm volatile("" : "+v"(zero));                 // (not a vector of zeros in registers of its own)
#pragma unroll
    for (int s = 0; s < FB; ++s)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[s][e] = zero;

    // ---- the weights of up to 64 records in a row at hand, in LDS ----
    v4f *wlds = lds4 + wave * kBatch;
    const uint32_t wa = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(wlds));
    uint32_t kb = 0;
    auto fetch_batch = [&](uint32_t k) {
        kb = k;
        const int ln = fresh_lane();
        const float4 w = a.w4[min(k + uint32_t(ln), a.n_records)];
        wlds[ln] = v4f{w.x, w.y, w.z, w.w};
    };
    fetch_batch(k_lo);
    uint32_t word0 = meta[now.record], word1 = meta[now.record + 1];           // (the stream is padded)
    // the registers of the record loop
    v16f in0, in1;
    v4f in2;
    if (SUB2) {                                    // (what is never read has to have a value)
        rows[5] = v4f{zero, zero, zero, zero};
#pragma unroll
        for (int e = 0; e < 16; ++e) in1[e] = zero;
        in2 = rows[5];
    }
    for (int left = n_visits; left > 0; --left) {
        const uint32_t k = now.record, k_end = k + (now.channel_count >> 16);
        // the lane's 6x6 neighbourhood, in the order of the record loop's registers
        float l[6], r6[6];
        {
            const uint32_t maskl = mask(0), maskr = mask(1);
            float from_l[6], from_r[6];
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                from_l[r] = rows[r][3]; from_r[r] = rows[r][0];
                if (OVER > 0) {
                    const uint32_t give_l = mask(2), give_r = mask(3);
                    from_l[r] = __uint_as_float((__float_as_uint(rows[r][3 - OVER]) & give_l) | (__float_as_uint(from_l[r]) & ~give_l));
                    from_r[r] = __uint_as_float((__float_as_uint(rows[r][OVER]) & give_r) | (__float_as_uint(from_r[r]) & ~give_r));
                }
            }
            // (lane 0 and lane 63 have nothing to read: zero, or see below; a lane shift may read a
            // register that a vector instruction wrote only after two more instructions)
#define PCONV_SHIFT(to, from, mask, way) "v_and_b32_dpp %" #to ", %" #from ", %" #mask " " way ":1 row_mask:0xf bank_mask:0xf bound_ctrl:0\n"
            if constexpr (SUB2)
                asm("s_nop 1\n"
                    PCONV_SHIFT(0, 5, 10, "wave_shr") PCONV_SHIFT(1, 6, 10, "wave_shr") PCONV_SHIFT(2, 7, 10, "wave_shr")
                    PCONV_SHIFT(3, 8, 10, "wave_shr") PCONV_SHIFT(4, 9, 10, "wave_shr")
                    : "=&v"(l[0]), "=&v"(l[1]), "=&v"(l[2]), "=&v"(l[3]), "=&v"(l[4])
                    : "v"(from_l[0]), "v"(from_l[1]), "v"(from_l[2]), "v"(from_l[3]), "v"(from_l[4]), "v"(maskl));
            else
            asm("s_nop 1\n"
                PCONV_SHIFT(0, 12, 24, "wave_shr") PCONV_SHIFT(1, 13, 24, "wave_shr") PCONV_SHIFT(2, 14, 24, "wave_shr")
                PCONV_SHIFT(3, 15, 24, "wave_shr") PCONV_SHIFT(4, 16, 24, "wave_shr") PCONV_SHIFT(5, 17, 24, "wave_shr")
                PCONV_SHIFT(6, 18, 25, "wave_shl") PCONV_SHIFT(7, 19, 25, "wave_shl") PCONV_SHIFT(8, 20, 25, "wave_shl")
                PCONV_SHIFT(9, 21, 25, "wave_shl") PCONV_SHIFT(10, 22, 25, "wave_shl") PCONV_SHIFT(11, 23, 25, "wave_shl")
                : "=&v"(l[0]), "=&v"(l[1]), "=&v"(l[2]), "=&v"(l[3]), "=&v"(l[4]), "=&v"(l[5]),
                  "=&v"(r6[0]), "=&v"(r6[1]), "=&v"(r6[2]), "=&v"(r6[3]), "=&v"(r6[4]), "=&v"(r6[5])
                : "v"(from_l[0]), "v"(from_l[1]), "v"(from_l[2]), "v"(from_l[3]), "v"(from_l[4]), "v"(from_l[5]),
                  "v"(from_r[0]), "v"(from_r[1]), "v"(from_r[2]), "v"(from_r[3]), "v"(from_r[4]), "v"(from_r[5]),
                  "v"(maskl), "v"(maskr));
#undef PCONV_SHIFT
            if (CUT) {
                const uint32_t mask0 = mask(4), mask63 = mask(5);
#pragma unroll
                for (int r = 0; r < (SUB2 ? 5 : 6); ++r) {
                    l[r] = __uint_as_float(__float_as_uint(l[r]) | (uint32_t(__builtin_amdgcn_readlane(__float_as_int(outer), 2 * r)) & mask0));
                    if (!SUB2) r6[r] = __uint_as_float(__float_as_uint(r6[r]) | (uint32_t(__builtin_amdgcn_readlane(__float_as_int(outer), 2 * r + 1)) & mask63));
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) in0[e] = rows[e >> 2][e & 3];
#pragma unroll
        for (int e = 0; e < (SUB2 ? 4 : 8); ++e) in1[e] = rows[4 + (e >> 2)][e & 3];
#pragma unroll
        for (int e = 0; e < (SUB2 ? 5 : 6); ++e) in1[8 + e] = l[e];
        if (!SUB2) {
            in1[14] = r6[0]; in1[15] = r6[1];
#pragma unroll
            for (int e = 0; e < 4; ++e) in2[e] = r6[2 + e];
        }
        // (a visit has at most 36 records: four kernels of nine taps)
        if (k < kb || k_end > kb + kBatch) fetch_batch(k);
#define PCONV_RECORD_LOOP_OPERANDS \
                : "+{v[64:79]}"(acc[0]), "+{v[80:95]}"(acc[1]), "+{v[96:111]}"(acc[2]), "+{v[112:127]}"(acc[3]), \
                  "+{v[28:43]}"(in0), "+{v[44:59]}"(in1), "+{v[60:63]}"(in2) \
                : [w0] "s"(word0 & ~kMetaFirstOfChannel), [w1] "s"(word1), [va] "v"(beside), \
                  [wa] "s"(wa + (k - kb) * 16u), [mp] "s"(a.meta), [koff] "s"(k * 4u), [nb] "s"(k_end - k), [chmask] "n"(0) \
                : "v22", "v23", "v24", "v25", "v26", "v27", \
                  "s84", "s85", "s86", "s90", "s91", "s92", "s93", "s94", "s95", "scc", "memory"
        if constexpr (SUB2)
            asm volatile(
#include "pconv_tiled_compute_scalar_sub2.inc"
                PCONV_RECORD_LOOP_OPERANDS);
        else
            asm volatile(
#include "pconv_tiled_compute_scalar.inc"
                PCONV_RECORD_LOOP_OPERANDS);
#undef PCONV_RECORD_LOOP_OPERANDS
        if (left == 1) break;
        // the input registers are free: the next channel, and what is needed to know the one after it
        load_rows(int(next.channel_count & 0xFFFFu));
        now = next;
        v = after(v);
        next = visit_at(after(v));
        word0 = meta[now.record]; word1 = meta[now.record + 1];
    }

    // ---- the partial sums are added through LDS, two slots at a time, and stored ----
    // Every wave that may have had channels writes its sums of two slots; then wave (u, i) adds up row i of the
    // patches in slot u, in order of the waves, and stores it (fused max-pool: rows 2 i and 2 i + 1).
    v4f *red = lds4 + NW * kBatch;                 // (behind the weights: nobody waits for the last wave's records)
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    const Patch patch = patch_of(lane_e);
    const int n = patch.n, y0 = patch.y0, x0 = patch.x0;
    if constexpr (SUB2) {
        // four outputs of a patch, all slots at once: wave s adds up slot s
        if (wave < parts) {
#pragma unroll
            for (int k = 0; k < FB; ++k)
                if (half < 0 || (k >> 1) == half) red[(wave * FB + k) * 64 + lane] = v4f{acc[k][0], acc[k][2], acc[k][8], acc[k][10]};
        }
        __syncthreads();
        if (wave >= FB || (half >= 0 && (wave >> 1) != half) || filter[0] < 0 || !patch.valid) return;
        v4f sum = red[wave * 64 + lane];
#pragma unroll 8
        for (int p = 1; p < parts; ++p) sum += red[(p * FB + wave) * 64 + lane];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            sum[k] += slot_bias[0];
            if (a.relu) sum[k] = fmaxf(sum[k], 0.0f);
        }
        const int h2 = (a.h + 1) >> 1, w2 = a.w >> 1;
        float *dst = a.y + ((size_t(n) * a.c_out + filter[0]) * h2 + (y0 >> 1)) * w2 + (x0 >> 1);
        dst[0] = sum[0]; dst[1] = sum[1];
        if (y0 + 2 < a.h) { dst[w2] = sum[2]; dst[w2 + 1] = sum[3]; }
        return;
    }
    auto store_rows = [&](int k, int u) {
        if (wave >= 8 || (a.pool && i >= 2) || (a.sub2 && (i & 1)) || !patch.valid) return;
        const int f = filter[k];
        if (f < 0) return;
        const float b = slot_bias[k];
        auto sum_row = [&](int row) {
            v4f sum = red[(u * 4 + row) * 64 + lane];
#pragma unroll 8
            for (int p = 1; p < parts; ++p) sum += red[((p * 2 + u) * 4 + row) * 64 + lane];
            return sum;
        };
        auto finish = [&](float v) { v += b; return a.relu ? fmaxf(v, 0.0f) : v; };
        if (a.pool) {
            const int hp = a.h >> 1, wp = a.w >> 1;
            const v4f t = sum_row(2 * i), q = sum_row(2 * i + 1);
            if ((y0 >> 1) + i >= hp) return;
            float *dst = a.y + ((size_t(n) * a.c_out + f) * hp + (y0 >> 1) + i) * wp + (x0 >> 1);
            *reinterpret_cast<float2 *>(dst) = make_float2(finish(fmaxf(fmaxf(t[0], t[1]), fmaxf(q[0], q[1]))),
                                                           finish(fmaxf(fmaxf(t[2], t[3]), fmaxf(q[2], q[3]))));
            return;
        }
        const v4f s = sum_row(i);
        if (y0 + i >= a.h) return;
        if (a.sub2) {
            // of the row the even columns (the patch starts at a multiple of 4, or at w - 4)
            const int h2 = (a.h + 1) >> 1, w2 = (a.w + 1) >> 1, k0 = x0 & 1;
            if (LAST) {
                float *dst = a.y + ((size_t(n) * h2 + ((y0 + i) >> 1)) * w2 + ((x0 + k0) >> 1)) * a.c_out + f;
                dst[0] = finish(k0 ? s[1] : s[0]);
                if (((x0 + k0) >> 1) + 1 < w2) dst[a.c_out] = finish(k0 ? s[3] : s[2]);
                return;
            }
            float *dst = a.y + ((size_t(n) * a.c_out + f) * h2 + ((y0 + i) >> 1)) * w2 + ((x0 + k0) >> 1);
            dst[0] = finish(k0 ? s[1] : s[0]);
            if (((x0 + k0) >> 1) + 1 < w2) dst[1] = finish(k0 ? s[3] : s[2]);
            return;
        }
        if (LAST) {
            float *dst = a.y + ((size_t(n) * a.h + y0 + i) * a.w + x0) * a.c_out + f;
#pragma unroll
            for (int k = 0; k < 4; ++k) dst[size_t(k) * a.c_out] = finish(s[k]);
            return;
        }
        float *dst = a.y + ((size_t(n) * a.c_out + f) * a.h + y0 + i) * a.w + x0;
        *reinterpret_cast<float4 *>(dst) = make_float4(finish(s[0]), finish(s[1]), finish(s[2]), finish(s[3]));
    };
#pragma unroll
    for (int pass = 0; pass < FB / 2; ++pass) {
        if (half >= 0 && pass != half) continue;
        if (pass > 0 && half < 0) __syncthreads(); // the pass before is done with
        if (wave < parts) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const v16f &s = acc[2 * pass + u];
                    red[((wave * 2 + u) * 4 + i) * 64 + lane] = v4f{s[4 * i], s[4 * i + 1], s[4 * i + 2], s[4 * i + 3]};
                }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER_PASS; ++k) store_rows(pass * PER_PASS + k, NW < 8 ? k : u);
    }
}

template <int OVER, bool CUT, bool LAST, int NW, bool SUB2 = false>
hipError_t launch_lone(const LoneArgs &a, unsigned wgs, hipStream_t st, int dev)
{
    constexpr size_t kLdsBytes = size_t(NW) * (kBatch + 2 * 4 * 64) * 16;   // weights and sums of two slots of every wave: 144 KB for 16
    // More dynamic LDS than the default limit: raised once per device (the flag is set to the same
    // value by every thread that gets here first).
    static std::atomic<bool> attr_done[64];
    if (dev < 0 || dev >= 64 || !attr_done[dev].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_lone_kernel<OVER, CUT, LAST, NW, SUB2>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, int(kLdsBytes));
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_done[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((conv_lone_kernel<OVER, CUT, LAST, NW, SUB2>), dim3(wgs), dim3(NW * 64), kLdsBytes, st, a);
    return hipGetLastError();
}

}  // namespace

// Whole rows of patches, unless that takes so many more rounds over the compute units that the outer columns,
// which make a visit a sixth longer (seven loads for six, 24 moves between lanes), are less.
LoneTiles lone_tiles(int64_t patches, int px, int64_t patch_base, int64_t groups, int slots)
{
    const int64_t left = patches - patch_base;
    const int rows = 64 / px;                      // whole patch rows of a tile
    LoneTiles t{64, true, (left + 63) / 64};
    if (rows > 0 && patch_base % px == 0) {
        const int64_t whole = (left + rows * px - 1) / (rows * px);
        auto rounds = [&](int64_t tiles) { return (tiles * groups + slots - 1) / slots; };
        if (rounds(whole) * 6 <= rounds(t.tiles) * 7) t = LoneTiles{rows * px, false, whole};
    }
    return t;
}

hipError_t launch_conv_lone(const pconv_handle *h, const float *x, float *y, const float *bias, int n, int hin, int win,
                            int stride, int relu, int pool, bool halves, int waves, int64_t patch_base, bool last, void *stream)
{
    LoneArgs a;
    a.x = x; a.y = y; a.bias = bias;
    a.slot_filter = h->d_slot_filter; a.bounds = h->d_lone_bounds; a.visits = h->d_lone_visits; a.meta = h->d_meta;
    a.w4 = reinterpret_cast<const float4 *>(h->d_w4);
    a.c_in = h->c_in; a.h = hin; a.w = win; a.c_out = h->c_out;
    a.px = (win + 3) / 4;
    a.per_img = (hin + 3) / 4 * a.px;
    a.n_patches = n * a.per_img; a.patch_base = int(patch_base);
    a.halves = halves;
    a.n_groups = h->tiled.num_blocks << (halves ? 1 : 0);
    const LoneTiles t = lone_tiles(a.n_patches, a.px, patch_base, a.n_groups, h->cus > 0 ? h->cus : 256);
    a.lanes = t.lanes;
    const int64_t units = t.tiles * a.n_groups;
    if (units > 0x3FFFFFFF) return hipErrorInvalidConfiguration;
    a.n_units = int(units);
    a.relu = relu; a.pool = pool; a.sub2 = stride == 2;
    a.n_records = uint32_t(h->tiled.meta.size()) - 3u;
    a.x_bytes = uint32_t(int64_t(n) * h->c_in * hin * win * 4);
    a.div_img = make_fast_div(uint32_t(a.per_img)); a.div_px = make_fast_div(uint32_t(a.px)); a.div_groups = make_fast_div(uint32_t(a.n_groups));
    const unsigned wgs = unsigned((units + 7) / 8 * 8);
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto launch = [&](auto over, auto cut) {
        constexpr int O = over.value;
        constexpr bool C = cut.value;
        if constexpr (O % 2 == 0)
            if (a.sub2 && !last)
                return waves == 16 ? launch_lone<O, C, false, 16, true>(a, wgs, st, h->device)
                       : waves == 8 ? launch_lone<O, C, false, 8, true>(a, wgs, st, h->device) : launch_lone<O, C, false, 4, true>(a, wgs, st, h->device);
        if (last)                                        // (16 waves only: see launch_conv_tiled)
            return launch_lone<O, C, true, 16>(a, wgs, st, h->device);
        return waves == 16 ? launch_lone<O, C, false, 16>(a, wgs, st, h->device)
               : waves == 8 ? launch_lone<O, C, false, 8>(a, wgs, st, h->device) : launch_lone<O, C, false, 4>(a, wgs, st, h->device);
    };
    auto launch_over = [&](auto over) { return t.cut ? launch(over, std::true_type{}) : launch(over, std::false_type{}); };
    switch (a.px * 4 - win) {
    case 0: return launch_over(std::integral_constant<int, 0>{});
    case 1: return launch_over(std::integral_constant<int, 1>{});
    case 2: return launch_over(std::integral_constant<int, 2>{});
    default: return launch_over(std::integral_constant<int, 3>{});
    }
}

}  // namespace pconv
