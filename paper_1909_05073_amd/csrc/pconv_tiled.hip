// Register-tiled PCONV kernel for gfx950 (stride 1; stride 2 at the same patches, of which the outputs at even rows
// and columns are stored: see SUB2).
//
// Work decomposition.  A workgroup of NW waves owns 64 "patches" (a patch = a 4x4 block of output
// pixels of one image; one patch per lane) and 4 * NW filters (4 per wave, its "slots").  Two shapes
// are built: 16 waves with 8-channel chunks (one workgroup fills a compute unit), and 8 waves with
// 4-channel chunks (two workgroups share a compute unit; used for layers with at most 4 input
// channels, where one workgroup's output stores overlap with the other's loads).  Either way a SIMD
// runs 4 waves: a single wave issues a vector instruction only about every 6.5 cycles, so it takes
// three to four of them to keep a SIMD busy.
//
// The input channels are walked in chunks of CH through two LDS buffers.  For a chunk, the 6x6 input
// neighbourhood of every patch is staged into LDS (zero outside the image, so the inner loops have
// no bounds tests) while the previous chunk is being computed, and every wave copies the weights
// of its records for the chunk into its own LDS block.  Then each wave walks its records: a
// record is one (kernel, code) pair, i.e. up to four kept taps of one 3x3 kernel of one of the
// wave's filters.  When a record starts a new input channel the lane reloads its 6x6 neighbourhood
// from LDS (nine 128-bit reads) and keeps it in registers for all of the wave's filters connected
// to that channel; the record itself costs 16 FMAs per kept tap on the slot's 16 accumulators.
//
// The record loop is generated assembly (gen_tiled_compute.py): the pattern of a kernel selects
// straight-line code with compile-time register indices (paper: per-pattern generated code, one
// branch per kernel instead of per weight), reached by one computed jump per record.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>

#include "pconv_internal.h"
#include "pconv_tiled_codes.h"

// Hand-over words for callers that cannot let the library allocate (pconv_conv2d_static): one row
// of kFlagWords words per device, in the code object itself.  Host code never uses this name as an
// address; it asks the runtime for the array's device address once per device (static_flags()).
static __device__ __align__(256) uint32_t scratch[pconv::kFlagWords];

namespace pconv {

namespace {

struct bf16_t { uint16_t bits; };

constexpr int FB = kTileFB, BATCH = kTileBatch;
// A staged channel is nine blocks of one 16-byte quad per patch: blocks 0-5 hold columns x0..x0+3
// of input rows y0-1..y0+4; blocks 6-8 hold the patch's twelve halo values e = 0..11 (quad e / 4,
// element e % 4): e < 6 is column x0-1 of row e, e >= 6 is column x0+4 of row e - 6.  A lane reads its
// whole 6x6 neighbourhood with nine 128-bit LDS reads.
constexpr int QUAD_FLOATS = 64 * 4;
constexpr int CHAN_FLOATS = 9 * QUAD_FLOATS;  // 2304
constexpr int ROWS_FLOATS = 6 * QUAD_FLOATS + 64;   // a channel of a wave on its own (PRIV)
constexpr int PLANE_FLOATS = ROWS_FLOATS + 4;       // the same with channels last: four planes on are 16 banks on
constexpr int INV_FLOATS = 2 * 64;            // per-lane invariants {offset, mask}
constexpr int SYNC_WORDS = 8;                 // counters that order the waves
constexpr int HALO_TAB_WORDS = 12 * 64;       // source offsets of the halo loads (VEC)

template <int NW, int CH> struct Shape {
    static constexpr int BUF_FLOATS = CH * CHAN_FLOATS;        // one chunk
    static constexpr int WLDS_FLOATS = NW * BATCH * 4;         // weight blocks of the waves
    static constexpr int OFF_W = 2 * BUF_FLOATS;
    static constexpr int OFF_INV = OFF_W + WLDS_FLOATS;
    static constexpr int OFF_SYNC = OFF_INV + INV_FLOATS;
    static constexpr int OFF_HALO = OFF_SYNC + SYNC_WORDS;
    // 16 waves x 8 channels: 159776 of the compute unit's 163840 bytes; 8 x 4: 81696 (two fit)
    static constexpr int OFF_OUT = OFF_HALO + HALO_TAB_WORDS;   // per wave: {filter, bias} of its four slots
    static constexpr size_t LDS_BYTES = size_t(OFF_OUT + NW * 2 * FB) * 4;
    static constexpr int UNITS = 2 * CH;                       // staging units of half a channel per chunk
    static constexpr int SEGS = CH * 6 / NW;                   // (channel, row) segments per wave (register path)
    static_assert(CH * 6 % NW == 0 && UNITS % 8 == 0 && CH <= kTileCH && kTileCH % CH == 0, "unsupported shape");
};

static_assert(FB == 4 && BATCH == 32 && kTileCH == 8,
              "gen_tiled_compute.py is written for 4 slots, 32-record batches, channel field of 3 bits");

__device__ __forceinline__ float ld_act(const float *p, size_t i) { return p[i]; }
__device__ __forceinline__ float ld_act(const bf16_t *p, size_t i) { return __uint_as_float(uint32_t(p[i].bits) << 16); }
__device__ __forceinline__ void st_act(float *p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void st_act(bf16_t *p, size_t i, float v)
{
    const uint32_t u = __float_as_uint(v);
    const uint32_t r = ((u & 0x7FFFFFFFu) > 0x7F800000u) ? ((u >> 16) | 0x40u) : ((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
    p[i].bits = uint16_t(r);
}

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
// Byte offset that lies beyond any tensor the VEC kernel accepts (at most 2^31 - 1 bytes): a buffer
// load at such an offset touches no memory and returns zero.
constexpr uint32_t kOutOfRange = 0x80000000u;

struct TiledArgs {
    const void *x; void *y; const float *bias;
    const int32_t *slot_filter; const uint32_t *chan_ptr; const uint32_t *meta; const float4 *w4;
    int n_img, c_in, row_len, h, w, c_out;
    int py, px;                 // patches per image column / row
    int n_patches, n_tiles, n_groups, n_blocks;
    int relu;
    int pool;                   // 1: y is the 2x2 / stride-2 max-pooled output (VEC kernel, whole units only)
    int sub2;                   // 1: stride 2: y holds the outputs at even rows and columns only
    int ks_log2;                // log2 of the channel split inside a workgroup (0, 1 or 2)
    int n_units;                // n_tiles * n_groups: (tile, filter group) pairs
    int n_chunks;               // chunks of CH input channels
    int split_units;            // 1: a workgroup's share of the work may begin and end inside a unit
    int priv;                   // 1: the 16 waves are 16 channel ranges of one filter block (channels last)
    int one_set;                // 1 (with split_units): the iterations are dealt over all workgroups as one set
    uint32_t *flags;            // [gridDim.x] hand-over words of this call (split_units only)
    uint32_t n_records;         // records of the stream (the padding record's index)
    uint32_t epoch;             // value that marks a hand-over word as set by this call (never 0)
    uint32_t x_bytes;           // size of the input tensor (VEC kernel: below 2^31)
    uint32_t y_bytes;           // size of the output tensor (shared units only: below 2^31)
    uint32_t *err;              // sticky error word of the handle (host memory the device can write)
    int spin_limit;             // iterations after which a wait inside the kernel gives up
};

// Error codes a kernel leaves in the handle's error word.
constexpr uint32_t kErrChunkWait = 1u, kErrHandOverWait = 2u;

template <typename T, int LAYOUT>
__device__ __forceinline__ size_t act_at(int n, int c, int y, int x, int C, int H, int W)
{
    if (LAYOUT == PCONV_NCHW) return ((size_t(n) * C + c) * H + y) * W + x;
    return ((size_t(n) * H + y) * W + x) * C + c;
}

// How the work is spread over the workgroups.  A unit is one (tile of 64 patches, group of 4 * FW
// filters) pair walked over all chunks of input channels; one unit step ("iteration") is one chunk
// of one unit.  The workgroups whose ids are equal mod 8 run on one XCD (one L2); set s gets one
// contiguous eighth of the tiles with all their filter groups, tile-major, so that the filter
// groups of a tile, and neighbouring tiles (which share input rows and columns), read their input
// through the same L2 at about the same time.  Inside a set the iterations are dealt out evenly:
//   split_units == 0   in whole units (a workgroup gets zero or more of them);
//   split_units == 1   as equal contiguous ranges of iterations, so a unit may be shared by two
//                      or more consecutive workgroups of the set, each taking a range of its chunks
//                      (with one_set: over all workgroups as a single set, whatever their XCD).
// The workgroups that share a unit add their partial sums through the output tensor itself, in
// order of their ids: each one adds what its predecessor left there, and either leaves the new
// sum for its successor (raw, no bias) or, if it holds the unit's last chunk, finishes the
// outputs.  A workgroup runs the piece it must hand on first and the piece it takes over last;
// the hardware starts workgroups in order of their ids, so whatever a workgroup waits for
// belongs to a workgroup that has already started and handed over at its very beginning.
//
//
// PRIV: few units of work, channels last (pconv_lone.hip does the same for NCHW, where a wave loads its
// channels by itself).  A workgroup is one filter block, its 16 waves are 16 ranges of channels, and the 16
// partial sums are added through LDS at the end.  The waves stage 16 channels together, four lanes to a
// pixel, and then run one each (128 channels @28, eight images: 33 us; with a lane per pixel 111, in whole
// units 118, with their channels split four ways 61).  The halo columns are not staged but read out of
// the neighbouring lanes' registers.
//
// VEC: fp32 NCHW tensors at least 4 wide move the four centre columns of a patch row (and the four
// outputs of a row) with one 128-bit access; the inputs go from global memory straight to LDS.
//
// SUB2: stride 2 with all patches starting at even columns (an even width): the record loop forms only the
// outputs that are stored, 16 FMAs a record instead of 64, and reads seven quads of a neighbourhood instead of
// nine.  What is left is the staging of every chunk, which a quarter of the FMAs no longer covers (128 channels
// @56, 16 images: 62.3 -> 55 us; the next record's weights asked for ahead of the FMAs change nothing, nor do
// two smaller workgroups per compute unit, 77).
template <typename T, int LAYOUT, bool VEC, int NW, int CH, bool SPLIT, bool PRIV = false, bool SUB2 = false>
__global__ void __launch_bounds__(NW * 64, 4)   // 4 waves per SIMD: at most 128 VGPRs
conv_tiled_kernel(const TiledArgs a)
{
    using S = Shape<NW, CH>;
    constexpr int BUF_FLOATS = S::BUF_FLOATS;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    // Everything outside the record loop (staging, the counters other waves wait for, the
    // epilogue) runs at the highest issue priority; the record loop drops to the lowest.
    __builtin_amdgcn_s_setprio(3);

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // The waves are FW filter blocks x KS channel splits (KS = 1 for large layers).  With KS > 1
    // the waves of one filter block share its filters, each takes CH / KS of the channels of every
    // chunk, and the partial sums are added through LDS at the end in a fixed order.
    const int ks_log2 = a.ks_log2;
    const int fw = NW >> ks_log2;                        // filter blocks per workgroup
    const int ksplit = wave / fw;                        // this wave's channel split
    const int chs = CH >> ks_log2;                       // channels of a chunk per split
    const int sub_lo = ksplit * chs, sub_hi = sub_lo + chs;

    const T *__restrict__ x = static_cast<const T *>(a.x);
    T *__restrict__ y = static_cast<T *>(a.y);
    const uint32_t lds_base = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
    // buffer resource of the input tensor (VEC staging): base, stride 0, size in bytes, raw 32-bit data
    v4u rsrc;
    {
        const uint64_t xa = reinterpret_cast<uint64_t>(a.x);
        rsrc.x = __builtin_amdgcn_readfirstlane(uint32_t(xa));
        rsrc.y = __builtin_amdgcn_readfirstlane(uint32_t(xa >> 32) & 0xFFFFu);
        rsrc.z = __builtin_amdgcn_readfirstlane(a.x_bytes);
        rsrc.w = 0x00020000u;
    }
    // (Per-lane values are deliberately recomputed where they are used, from a lane id the
    // compiler cannot see through: only a few vector registers may stay live across the record
    // loop, and a spill reload there would wait for the loads in flight for the next chunk.)
    auto fresh_lane = [&]() { int l = threadIdx.x & 63; asm volatile("" : "+v"(l)); return l; };
    float *wlds = lds + S::OFF_W + wave * (BATCH * 4);   // this wave's weight block
    const uint32_t wa = lds_base + uint32_t(S::OFF_W + wave * (BATCH * 4)) * 4u;
    int *inv = reinterpret_cast<int *>(lds + S::OFF_INV);
    unsigned *sync_words = reinterpret_cast<unsigned *>(lds + S::OFF_SYNC);
    int *halo_tab = reinterpret_cast<int *>(lds + S::OFF_HALO);
    const int per_img = a.py * a.px;
    const int hw = a.h * a.w;
    const int n_chunks = a.n_chunks;

    // ---- this workgroup's range of iterations ----
    // (one_set: no XCD sets - the shares of all workgroups are then equal whatever the number of tiles,
    // and the workgroup that a piece waits for is simply the one before it)
    const bool one_set = PRIV || (SPLIT && a.one_set);
    // (PRIV: XCD s gets the s-th eighth of the units, so that its L2 serves few tiles)
    const int per_xcd = PRIV ? (a.n_units + 7) >> 3 : 0;
    const int set = one_set ? 0 : int(blockIdx.x & 7);
    const int j_in_set = PRIV ? int(blockIdx.x & 7) * per_xcd + int(blockIdx.x >> 3) : one_set ? int(blockIdx.x) : int(blockIdx.x >> 3);
    const int set_stride = one_set ? 1 : 8;
    // set s: the contiguous block of tiles [s * tps, (s + 1) * tps): neighbouring tiles (which share
    // input rows and columns) then run next to each other in time on one XCD and find them in its L2
    // (with tiles s, s + 8, ... in a set, conv2 of VGG-16 fetched 699 MB for its 411 MB input; now 444)
    const int tps = (a.n_tiles + 7) >> 3;
    const int set_tile0 = set * tps;
    const int set_units = one_set ? a.n_units : max(0, min(a.n_tiles, set_tile0 + tps) - set_tile0) * a.n_groups;
    // SPLIT: iteration = (unit of the set) * n_chunks + chunk; otherwise one whole unit per workgroup
    int ua = j_in_set, ub = j_in_set, head_c0 = 0, tail_c1 = n_chunks;
    if constexpr (SPLIT) {
        const int wgs_in_set = one_set ? int(gridDim.x) : (int(gridDim.x) - set + 7) >> 3;
        const int64_t iters = int64_t(set_units) * n_chunks;
        const int64_t takers = iters < wgs_in_set ? iters : wgs_in_set;       // nobody gets an empty range in between
        if (j_in_set >= takers) return;
        int64_t it0 = iters * j_in_set / takers, it1 = iters * (j_in_set + 1) / takers;
        // When every unit is shared by the same number P of workgroups, those finish their chunks at
        // the same time and then pass the sums on one after the other, each link of that chain taking
        // about as long as 2.5 chunks.  Their shares are therefore graded, the first the smallest and
        // 2.5 chunks more for each successor (boundary k at k n / P - 2.5 k (P - k) / 2), so that a
        // workgroup finishes about when its predecessor's sums arrive.
        const int P = int(takers / set_units);
        if (set_units * P == takers && P >= 2 && 4 * n_chunks >= P * (16 + 5 * (P - 1))) {
            const int u = j_in_set / P, kk = j_in_set - u * P;
            auto bound = [&](int q) { return (4 * q * n_chunks / P - 5 * q * (P - q)) / 4; };
            it0 = int64_t(u) * n_chunks + bound(kk);
            it1 = int64_t(u) * n_chunks + bound(kk + 1);
        }
        ua = int(it0 / n_chunks); ub = int((it1 - 1) / n_chunks);            // first and last unit touched
        head_c0 = int(it0 - int64_t(ua) * n_chunks);                         // > 0: unit ua begins elsewhere
        tail_c1 = int(it1 - int64_t(ub) * n_chunks);                         // < n_chunks: unit ub ends elsewhere
    } else {
        if (j_in_set >= set_units || (PRIV && int(blockIdx.x >> 3) >= per_xcd)) return;
    }
    const bool has_head = head_c0 > 0, has_tail = tail_c1 < n_chunks;
    const bool one_piece = ua == ub;
    // order: the piece to hand on, whole units, the piece taken over
    const int first_whole = has_head ? ua + 1 : ua, last_whole = has_tail ? ub - 1 : ub;
    const int n_whole = last_whole >= first_whole ? last_whole - first_whole + 1 : 0;
    const int n_pieces = SPLIT ? (has_tail ? 1 : 0) + n_whole + ((has_head && !(one_piece && has_tail)) ? 1 : 0) : 1;

    for (int piece = 0; piece < n_pieces; ++piece) {
        int unit, c_begin = 0, c_end = n_chunks;
        if (has_tail && piece == 0) { unit = ub; c_end = tail_c1; if (one_piece) c_begin = head_c0; }
        else if (piece - (has_tail ? 1 : 0) < n_whole) unit = first_whole + piece - (has_tail ? 1 : 0);
        else { unit = ua; c_begin = head_c0; }
        const bool takes_over = SPLIT && c_begin > 0, hands_on = SPLIT && c_end < n_chunks;
        const int tile = (one_set ? 0 : set_tile0) + unit / a.n_groups, group = unit % a.n_groups;
        const int fblk = PRIV ? group : group * fw + (wave - ksplit * fw);
        const bool active = fblk < a.n_blocks;

        if (SPLIT) __syncthreads();                      // every wave has left the previous piece: LDS is free

        // The records of a (filter block, chunk) are contiguous and ordered by channel, so this wave's
        // share of a chunk is the range between two entries of chan_ptr.  The range bounds of up to
        // 64 consecutive chunks sit one per lane in ptr_pk and are read with v_readlane.
        // (Loaded first: they are on the way while the tables below are set up.)
        const int ptr_max = a.row_len - 1;               // last entry of a row: end of the block's records
        const uint32_t *__restrict__ ptr_row = a.chan_ptr + size_t(active ? fblk : 0) * a.row_len;
        int win_base = c_begin;
        // one register holds both bounds: first record (24 bits) and number of records (8 bits)
        auto load_bounds = [&]() {
            const uint32_t lo = ptr_row[min((win_base + lane) * CH + sub_lo, ptr_max)];
            const uint32_t hi = ptr_row[min((win_base + lane) * CH + sub_hi, ptr_max)];
            return lo << 8 | (hi - lo);
        };
        uint32_t ptr_pk = load_bounds();
        // The epilogue needs each slot's filter index and bias: two dependent loads, started here and
        // parked in LDS so that they cost the epilogue nothing (and no registers in between).
        float *out_tab = lds + S::OFF_OUT + wave * (2 * FB);
        if (lane < FB) {
            const int f = active ? a.slot_filter[fblk * FB + lane] : -1;
            const float b = (a.bias && f >= 0) ? a.bias[f] : 0.0f;
            out_tab[2 * lane] = __int_as_float(f);
            out_tab[2 * lane + 1] = b;
        }


        // this lane's patch
        const int pidx = tile * 64 + lane;
        const bool pvalid = pidx < a.n_patches;
        const int n = pvalid ? pidx / per_img : 0;
        const int prem = pvalid ? pidx - n * per_img : 0;
        // VEC: the last patch of a row is shifted left so that it ends at the image edge: the four
        // centre columns of a patch row are then always inside the image.  It overlaps its neighbour, and
        // both store the shared columns, also from two workgroups where a tile ends between them: the
        // order of the additions must not depend on the tile (in every form of a launch it follows
        // from the filter; a second launch for the last tiles comes after the first one's stores).
        const int y0 = (prem / a.px) * 4;
        const int x0 = VEC ? min((prem % a.px) * 4, a.w - 4) : (prem % a.px) * 4;

        // accumulators: slot s, output (row i, column k) of the patch = acc[s][4 * i + k].  The record
        // loop is assembly with a fixed register map, so each vector is pinned to its registers there.
        v16f acc[FB];
#pragma unroll
        for (int s = 0; s < FB; ++s) acc[s] = 0.0f;

        // ---- staging ----
        // Loads are branch-free: an out-of-image element is not loaded (VEC) or reads element 0 of the
        // tensor and is replaced by zero when the segment is written to LDS.  What is valid for this
        // lane does not change from chunk to chunk and is kept as one bit mask: bits 0-5 input rows
        // y0-1 .. y0+4, bits 8-13 input columns x0-1 .. x0+4.
        uint32_t vmask0 = 0;
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const int iy = y0 - 1 + r, ix = x0 - 1 + r;
            if (pvalid && iy >= 0 && iy < a.h) vmask0 |= 1u << r;
            if (ix >= 0 && ix < a.w) vmask0 |= 0x100u << r;
        }
        // element offset of (channel 0 of the chunk, row y0-1, column x0) follows from c0; tensors have
        // fewer than 2^31 elements, so 32-bit offsets suffice (they are only used where valid)
        const int lane_off0 = LAYOUT == PCONV_NCHW ? (n * a.c_in * a.h + (y0 - 1)) * a.w + x0
                                                  : ((n * a.h + (y0 - 1)) * a.w + x0) * a.c_in;
        // all waves work on the same 64 patches: the per-lane invariants live in LDS, one copy
        if (threadIdx.x < SYNC_WORDS) sync_words[threadIdx.x] = 0;
        if (wave == 0) { inv[2 * lane] = lane_off0; inv[2 * lane + 1] = int(vmask0); }
        // VEC path: the twelve halo values of a patch are fetched by twelve one-word loads per channel,
        // each of which fills 64 consecutive words of the halo blocks: word i of load j belongs to patch
        // 16 * (j % 4) + i / 4 and is its halo value e = 4 * (j / 4) + i % 4.  The element offset of that
        // value in channel 0, in bytes (or kOutOfRange outside the image), is the same for every chunk: tabulated once.
        if (VEC) {
            for (int t = threadIdx.x; t < HALO_TAB_WORDS; t += NW * 64) {
                const int j = t >> 6, i = t & 63;
                const int e = 4 * (j >> 2) + (i & 3);
                const int pidx_h = tile * 64 + 16 * (j & 3) + (i >> 2);
                const int n_h = pidx_h / per_img, prem_h = pidx_h - n_h * per_img;
                const int iy = (prem_h / a.px) * 4 - 1 + (e < 6 ? e : e - 6);
                const int xh = min((prem_h % a.px) * 4, a.w - 4);
                const int ix = e < 6 ? xh - 1 : xh + 4;
                const bool ok = pidx_h < a.n_patches && iy >= 0 && iy < a.h && ix >= 0 && ix < a.w;
                halo_tab[t] = ok ? ((n_h * a.c_in * a.h + iy) * a.w + ix) * 4 : int(kOutOfRange);
            }
        }
        // VEC path: global -> LDS directly, no registers and next to no vector ALU work.  The LDS
        // words of rows and halo values outside the image are zeroed once per piece and never get
        // anything but zero, so they stay zero for every chunk.
        // One unit of staging work = half a channel: three rows and six halo loads.
        auto stage_direct = [&](int c0, float *buf, int sunit) {
            const int ln = fresh_lane();
            const int ch = sunit >> 1, half = sunit & 1;
            if (c0 + ch >= a.c_in) return;                               // (uniform)

            const uint32_t soff = __builtin_amdgcn_readfirstlane(uint32_t(c0 + ch) * uint32_t(hw) * 4u);
            float *cbuf = buf + ch * CHAN_FLOATS;
            // everything the lane needs from the tables first, so that there is one wait for LDS
            const int lane_off_now = inv[2 * ln];
            const uint32_t vmask = uint32_t(inv[2 * ln + 1]);
            uint32_t off[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) off[k] = uint32_t(halo_tab[(6 * half + k) * 64 + ln]);
            // Buffer loads: address = tensor + soff (channel, uniform) + per-lane byte offset; a lane
            // whose row or halo value lies outside the image has an offset beyond the buffer's size,
            // for which the hardware reads nothing and delivers zero.  The LDS address of lane 0's
            // element goes to M0 and every lane adds lane * size.  Written as assembly so that the
            // compiler does not track these loads: it would otherwise wait for them before the record
            // loop (they are waited for explicitly before they are published).
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int r = 3 * half + k;
                const uint32_t voff = ((vmask >> r) & 1u) ? uint32_t(lane_off_now + r * a.w) * 4u : kOutOfRange;
                const uint32_t dst_b = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(cbuf + r * QUAD_FLOATS));
                asm volatile("s_mov_b32 m0, %1\n s_nop 0\n buffer_load_dwordx4 %0, %2, %3 offen lds"
                             ::"v"(voff), "s"(dst_b), "s"(rsrc), "s"(soff));
            }
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                const int j = 6 * half + k;
                const uint32_t dst_b = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(cbuf + 6 * QUAD_FLOATS + j * 64));
                asm volatile("s_mov_b32 m0, %1\n s_nop 0\n buffer_load_dword %0, %2, %3 offen lds"
                             ::"v"(off[k]), "s"(dst_b), "s"(rsrc), "s"(soff));
            }
        };
        // generic path (any layout / dtype / width): through registers, with conversion to fp32;
        // every thread owns SEGS (channel, row) segments of its lane's patch
        constexpr int SEGS = S::SEGS;
        auto stage_load = [&](int c0, float (&t)[SEGS][6]) {
            const int ln = fresh_lane();
            const int lane_off_now = inv[2 * ln];
            const uint32_t vmask = uint32_t(inv[2 * ln + 1]);
#pragma unroll
            for (int kk = 0; kk < SEGS; ++kk) {
                const int seg = wave + NW * kk;
                const int ch = seg / 6, r = seg - ch * 6;
                const bool rv = ((vmask >> r) & 1u) && (c0 + ch < a.c_in);
                const int off = LAYOUT == PCONV_NCHW ? lane_off_now + (c0 + ch) * hw + r * a.w
                                                     : lane_off_now + r * a.w * a.c_in + (c0 + ch);
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) {
                    const bool ok = rv && ((vmask >> (8 + cc)) & 1u);
                    const int e = LAYOUT == PCONV_NCHW ? off + (cc - 1) : off + (cc - 1) * a.c_in;
                    t[kk][cc] = ld_act(x, size_t(ok ? e : 0));
                }
            }
        };
        auto stage_store = [&](int c0, float *buf, const float (&t)[SEGS][6]) {
            const int ln = fresh_lane();
            const uint32_t vmask = uint32_t(inv[2 * ln + 1]);
#pragma unroll
            for (int kk = 0; kk < SEGS; ++kk) {
                const int seg = wave + NW * kk;
                const int ch = seg / 6, r = seg - ch * 6;
                const bool rv = ((vmask >> r) & 1u) && (c0 + ch < a.c_in);
                float v[6];
#pragma unroll
                for (int cc = 0; cc < 6; ++cc) v[cc] = (rv && ((vmask >> (8 + cc)) & 1u)) ? t[kk][cc] : 0.0f;
                float *cbuf = buf + ch * CHAN_FLOATS;
                *reinterpret_cast<float4 *>(cbuf + r * QUAD_FLOATS + ln * 4) = make_float4(v[1], v[2], v[3], v[4]);
                cbuf[(6 + r / 4) * QUAD_FLOATS + ln * 4 + r % 4] = v[0];                    // halo value e = r
                cbuf[(6 + (6 + r) / 4) * QUAD_FLOATS + ln * 4 + (6 + r) % 4] = v[5];        // halo value e = 6 + r
            }
        };
        // four consecutive channels of a pixel (channels last), element offset e, zero unless ok
        auto four = [&](bool ok, int e) {
            v4f v;
            if constexpr (sizeof(T) == 4) {
                __builtin_memcpy(&v, x + (ok ? e : 0), 16);
            } else {
                uint2 u;
                __builtin_memcpy(&u, x + (ok ? e : 0), 8);
                v = v4f{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                        __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u)};
            }
            return ok ? v : v4f{0.f, 0.f, 0.f, 0.f};
        };
        // Channels last, c_in a multiple of 4: CH / 4 neighbouring lanes load the chunk's channels of a
        // pixel, an instruction 256 / CH pixels of one input row (one channel per wave and pixel column
        // per load, as in stage_load, touches a cache line per lane: 16 images @56 to 256 filters in whole
        // units, records included, 21.0 us a chunk with 254 channels, 10.1 with 256).  A pixel is
        // loaded once and also written to the halo words of the patch beside it; halo words outside
        // the image are never written and stay zero.
        auto stage_quads = [&](int c0, float *buf) {
            constexpr int QUADS = CH / 4, PIX = 64 / QUADS, GROUPS = 256 / PIX;
            static_assert(6 * GROUPS == SEGS * NW, "items per wave");
            const int ln = fresh_lane();
            const int quad = ln & (QUADS - 1), c4 = c0 + quad * 4;
            float *cbuf = buf + quad * 4 * CHAN_FLOATS;
            v4f v[SEGS], beside = v4f{0.f, 0.f, 0.f, 0.f};
            const int eb = ln / QUADS, rb = eb >> 1, pb = (eb & 1) ? 63 : 0;       // wave 0: beside the tile's first and last patch
#pragma unroll
            for (int i = 0; i < SEGS; ++i) {
                const int item = wave * SEGS + i, r = item / GROUPS, pix = (item % GROUPS) * PIX + ln / QUADS, patch = pix >> 2, q = pix & 3;
                const uint32_t vmask = uint32_t(inv[2 * patch + 1]);
                const bool ok = ((vmask >> r) & (vmask >> (9 + q)) & 1u) && c4 < a.c_in;
                v[i] = four(ok, inv[2 * patch] + (r * a.w + q) * a.c_in + c4);
            }
            if (wave == 0 && eb < 12) {
                const uint32_t vmask = uint32_t(inv[2 * pb + 1]);
                const bool ok = ((vmask >> rb) & (vmask >> (pb ? 13 : 8)) & 1u) && c4 < a.c_in;
                beside = four(ok, inv[2 * pb] + (rb * a.w + (pb ? 4 : -1)) * a.c_in + c4);
            }
#pragma unroll
            for (int i = 0; i < SEGS; ++i) {
                const int item = wave * SEGS + i, r = item / GROUPS, pix = (item % GROUPS) * PIX + ln / QUADS, patch = pix >> 2, q = pix & 3;
                const uint32_t vmask = uint32_t(inv[2 * patch + 1]);
                // halo value e of a patch lies at word 4 * patch + e % 4 of block 6 + e / 4
                int halo = -1;
                if (q == 3 && ((vmask >> 13) & 1u) && patch < 63) halo = (6 + r / 4) * QUAD_FLOATS + (patch + 1) * 4 + r % 4;
                if (q == 0 && ((vmask >> 8) & 1u) && patch > 0) halo = (6 + (6 + r) / 4) * QUAD_FLOATS + (patch - 1) * 4 + (6 + r) % 4;
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    cbuf[k4 * CHAN_FLOATS + r * QUAD_FLOATS + pix] = v[i][k4];
                    if (halo >= 0) cbuf[k4 * CHAN_FLOATS + halo] = v[i][k4];
                }
            }
            if (wave == 0 && eb < 12) {
                const int e = pb ? 6 + rb : rb;
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) cbuf[k4 * CHAN_FLOATS + (6 + e / 4) * QUAD_FLOATS + pb * 4 + e % 4] = beside[k4];
            }
        };
        // (rel = chunk index relative to the piece; it selects the LDS buffer)
        auto stage = [&](int rel) {
            if constexpr (LAYOUT == PCONV_NHWC)
                if (a.c_in % 4 == 0) { stage_quads((c_begin + rel) * CH, lds + (rel & 1) * BUF_FLOATS); return; }
            float t[SEGS][6];
            stage_load((c_begin + rel) * CH, t);
            stage_store((c_begin + rel) * CH, lds + (rel & 1) * BUF_FLOATS, t);
        };

        if (VEC || LAYOUT == PCONV_NHWC) {
            // zero both staged buffers (see stage_direct, stage_quads)
#pragma unroll
            for (int j = 0; j < 2 * BUF_FLOATS / (NW * 64 * 4); ++j)
                *reinterpret_cast<float4 *>(lds + (j * NW * 64 + threadIdx.x) * 4) = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();                                 // zeroed buffers, tables and counters are visible

        // record range of this wave for a chunk, and the fetch of its first batch: lane j gets record
        // j (k0 + k_cnt is the next record or the padding record, always readable)
        auto fetch_records = [&](int chunk, uint32_t &k0, uint32_t &k_cnt, uint32_t &rec_m, float4 &rec_w) {
            if (chunk - win_base > 63) {                 // every 64 chunks: next window of bounds
                win_base = chunk;
                ptr_pk = load_bounds();
                __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0) here, so that the common path needs no wait
            }
            const uint32_t pk = __builtin_amdgcn_readlane(ptr_pk, chunk - win_base);
            k0 = pk >> 8;
            k_cnt = active ? pk & 0xFFu : 0u;

            const uint32_t ridx = k0 + min(uint32_t(lane), k_cnt);
            rec_m = a.meta[ridx];
            rec_w = a.w4[ridx];
        };

        // ---- the records of one chunk: generated assembly, in batches of up to BATCH records ----
        auto compute = [&](int rel, uint32_t k0, uint32_t k_cnt, uint32_t rec_m) {
            const uint32_t buf_bytes = uint32_t(rel & 1) * uint32_t(BUF_FLOATS * 4);
            // (one loop around a single copy of the assembly: the refill of a further batch sits behind it)
            uint32_t base = 0;
            while (base < k_cnt) {
                const uint32_t nb = __builtin_amdgcn_readfirstlane(min(uint32_t(BATCH), k_cnt - base));
                // lane j = record j of the batch; the lanes behind the last record end the list
                const uint32_t rm = uint32_t(fresh_lane()) < nb ? rec_m : kMetaEndOfList;
                const uint32_t koff = __builtin_amdgcn_readfirstlane((k0 + base) * 4u);
#define PCONV_RECORD_LOOP_OPERANDS \
                    : "+{v[64:79]}"(acc[0]), "+{v[80:95]}"(acc[1]), "+{v[96:111]}"(acc[2]), "+{v[112:127]}"(acc[3]) \
                    : [recm] "v"(rm), [va] "v"(lds_base + buf_bytes + uint32_t(fresh_lane()) * 16u), \
                      [wa] "s"(wa), [mp] "s"(a.meta), [koff] "s"(koff), [nb] "s"(nb), [chmask] "n"(CH - 1) \
                    : "v22", "v23", "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", \
                      "v34", "v35", "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", \
                      "v46", "v47", "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", \
                      "v58", "v59", "v60", "v61", "v62", "v63", \
                      "s84", "s85", "s86", "s90", "s91", "s92", "s93", "s94", "s95", "scc"
                if constexpr (SUB2)
                    asm volatile(
#include "pconv_tiled_compute_sub2.inc"
                        PCONV_RECORD_LOOP_OPERANDS);
                else
                    asm volatile(
#include "pconv_tiled_compute.inc"
                        PCONV_RECORD_LOOP_OPERANDS);
#undef PCONV_RECORD_LOOP_OPERANDS
                // No "memory" clobber on purpose: it would make the compiler wait for the
                // global->LDS loads of the next chunk, which may be in flight here and go to the
                // other buffer.  What the loop reads was published before (barrier / counters), or
                // written by the volatile stores below.
                base += BATCH;
                if (base < k_cnt) {
                    // more than BATCH records in this chunk (rare): next batch (the wave's weight
                    // block is private, and LDS accesses of one wave execute in order)
                    const uint32_t ridx = k0 + min(base + uint32_t(fresh_lane()), k_cnt);
                    rec_m = a.meta[ridx];
                    const float4 rec_w = a.w4[ridx];
                    // waiting here, in the rare path, keeps the common path free of a wait for all
                    // vector-memory loads (which would include the next chunk's staging)
                    __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0)
                    if (fresh_lane() == 0) rec_m |= kMetaFirstOfChannel;   // input registers do not survive between batches
                    if (fresh_lane() < BATCH) {
                        volatile float *wv = wlds + fresh_lane() * 4;
                        wv[0] = rec_w.x; wv[1] = rec_w.y; wv[2] = rec_w.z; wv[3] = rec_w.w;
                    }
                }
            }
        };

        uint32_t k0, k_cnt, rec_m;
        const int n_rel = c_end - c_begin;

        if constexpr (PRIV) {
            uint32_t kb = 0, kb_end = 0;                             // records whose words and weights are at hand
            uint32_t words = 0;
            // the lane's neighbourhood of the channel in slot `at` (bytes) to the registers of the record loop
            v16f in0, in1;
            v4f in2;
            auto load_patch = [&](uint32_t at) {
                const int ln = fresh_lane();
                // all ones where the column beside the patch lies in the image
                const uint32_t vmask = uint32_t(inv[2 * ln + 1]);
                const int maskl = int(vmask << 23) >> 31, maskr = int(vmask << 18) >> 31;
                asm volatile(
#include "pconv_tiled_patch_shifted.inc"
                    : "=&{v[28:43]}"(in0), "=&{v[44:59]}"(in1), "=&{v[60:63]}"(in2)
                    : [va] "v"(at + uint32_t(ln) * 16u), [further] "v"(at + uint32_t(6 * QUAD_FLOATS * 4) + uint32_t(ln) * 4u),
                      [maskl] "v"(maskl), [maskr] "v"(maskr)
                    : "v24", "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79");
            };
            // words and weights of the next BATCH records (index at most that of the padding record)
            auto fetch_batch = [&](uint32_t k, float4 &rec_w) {
                kb = k; kb_end = k + BATCH;
                const uint32_t ridx = min(k + uint32_t(fresh_lane() & (BATCH - 1)), a.n_records);
                words = a.meta[ridx];
                rec_w = a.w4[ridx];
            };
            auto store_batch = [&](const float4 &rec_w) {
                if (fresh_lane() < BATCH) {
                    volatile float *wv = wlds + fresh_lane() * 4;
                    wv[0] = rec_w.x; wv[1] = rec_w.y; wv[2] = rec_w.z; wv[3] = rec_w.w;
                }
            };
            auto run_records = [&](uint32_t k, uint32_t k_end) {
                while (k < k_end) {
                    if (k_end > kb_end || k < kb) {
                        float4 rec_w;
                        fetch_batch(k, rec_w);
                        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
                        store_batch(rec_w);
                    }
                    const uint32_t nb = min(k_end, kb_end) - k;
                    const uint32_t w0 = __builtin_amdgcn_readlane(words, k - kb) & ~kMetaFirstOfChannel;
                    const uint32_t w1 = __builtin_amdgcn_readlane(words, min(k + 1 - kb, uint32_t(BATCH - 1)));
                    asm volatile(
#include "pconv_tiled_compute_scalar.inc"
                        : "+{v[64:79]}"(acc[0]), "+{v[80:95]}"(acc[1]), "+{v[96:111]}"(acc[2]), "+{v[112:127]}"(acc[3]),
                          "+{v[28:43]}"(in0), "+{v[44:59]}"(in1), "+{v[60:63]}"(in2)
                        : [w0] "s"(w0), [w1] "s"(w1), [va] "v"(0u),
                          [wa] "s"(wa + (k - kb) * 16u), [mp] "s"(a.meta), [koff] "s"(k * 4u), [nb] "s"(nb), [chmask] "n"(0)
                        : "v22", "v23", "v24", "v25", "v26", "v27",
                          "s84", "s85", "s86", "s90", "s91", "s92", "s93", "s94", "s95", "scc");
                    k += nb;
                }
            };
            const uint32_t slot_at = lds_base + uint32_t(wave) * uint32_t(PLANE_FLOATS * 4);
            // ---- channels last: the waves stage 16 channels together, then every wave runs one ----
            // (four channels of a pixel are one load, so a wave cannot stage one channel well)
            uint32_t first = 0, count = 0;                       // lane j: records of this wave's channel in step win + j
            const int steps = (a.c_in + NW - 1) / NW;
            for (int step = 0; step < steps; ++step) {
                if ((step & 63) == 0) {
                    const int c0 = min((step + fresh_lane()) * NW + wave, ptr_max);
                    first = ptr_row[c0];
                    count = ptr_row[min(c0 + 1, ptr_max)] - first;
                }
                const uint32_t k = __builtin_amdgcn_readlane(first, step & 63);
                const uint32_t k_end = k + __builtin_amdgcn_readlane(count, step & 63);
                float4 rec_w;
                fetch_batch(k, rec_w);
                // Four lanes load the 16 channels of a pixel (64 bytes in a row), an instruction 16
                // pixels of one input row: four patches.  96 such items (six rows of 64 patches) are
                // six per wave; wave 0 also loads the pixels beside the tile's first and last patch.
                // A lane's four channels go to four planes.
                const int ln = fresh_lane();
                const int c4 = step * NW + (ln & 3) * 4;         // (c_in is a multiple of 4)
                v4f px[6], beside = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const int pix = wave * 16 + (ln >> 2), patch = pix >> 2, q = pix & 3;   // row i
                    const int off = inv[2 * patch];
                    const uint32_t vmask = uint32_t(inv[2 * patch + 1]);
                    const bool ok = ((vmask >> i) & (vmask >> (9 + q)) & 1u) && c4 < a.c_in;
                    px[i] = four(ok, off + (i * a.w + q) * a.c_in + c4);
                }
                if (wave == 0 && ln < 48) {
                    const int e = ln >> 2, r = e >> 1, patch = (e & 1) ? 63 : 0;
                    const int off = inv[2 * patch];
                    const uint32_t vmask = uint32_t(inv[2 * patch + 1]);
                    const bool ok = ((vmask >> r) & (vmask >> ((e & 1) ? 13 : 8)) & 1u) && c4 < a.c_in;
                    beside = four(ok, off + (r * a.w + ((e & 1) ? 4 : -1)) * a.c_in + c4);
                }
                if (step > 0) __syncthreads();                   // every wave has read its channel of the step before
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int k4 = 0; k4 < 4; ++k4)
                        lds[((ln & 3) * 4 + k4) * PLANE_FLOATS + i * QUAD_FLOATS + wave * 16 + (ln >> 2)] = px[i][k4];
                if (wave == 0 && ln < 48) {
#pragma unroll
                    for (int k4 = 0; k4 < 4; ++k4) lds[((ln & 3) * 4 + k4) * PLANE_FLOATS + 6 * QUAD_FLOATS + (ln >> 2)] = beside[k4];
                }
                store_batch(rec_w);
                __syncthreads();
                if (k != k_end) {
                    load_patch(slot_at);
                    run_records(k, k_end);
                }
            }
        } else if constexpr (VEC) {
            // ---- no barrier in this loop: three counters per LDS buffer order the waves ----
            //   tickets  staging work asked for           (a chunk has UNITS units of half a channel)
            //   staged   staging units whose data landed  chunk r is readable when staged == UNITS * (r/2 + 1)
            //   done     waves that finished a chunk      chunk r's buffer may be refilled (with chunk
            //                                             r + 2) when done == NW * (r/2 + 1)
            // All counters only grow.  A wave that has finished chunk r stages what is left of chunk
            // r + 1 (once every wave is done with chunk r - 1, whose buffer it takes), then computes it:
            // waves may be one chunk apart, so a chunk costs a wave its own records, not the records of
            // the busiest wave, and the staging falls to the waves with the least to do.  The slowest
            // wave never waits for a faster one: whatever it needs has been, or can be, produced by
            // itself.  Waits are bounded (TiledArgs::spin_limit polls) so that a mistake here ends in an
            // error code and poisoned outputs, not in a hang.
            unsigned *tickets = sync_words, *staged = sync_words + 2, *done = sync_words + 4;
            // A wait that runs out marks the workgroup (every wave poisons its outputs with NaN in
            // the epilogue) and leaves a code in the handle's error word, which the next call on
            // the handle reports.
            auto wait_ge = [&](unsigned *p, unsigned target) {
                bool reached = false;
                for (int guard = 0; guard < a.spin_limit; ++guard) {
                    const unsigned v = __builtin_amdgcn_readfirstlane(
                        __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
                    if (v >= target) { reached = true; break; }
                    __builtin_amdgcn_s_sleep(4);
                }
                if (!reached && fresh_lane() == 0) {
                    __hip_atomic_store(&sync_words[6], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __hip_atomic_store(a.err, kErrChunkWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
            };
            // A wave asks for staging work once per chunk, with one atomic add of kClaim: the counter
            // of a buffer therefore advances by exactly NW * kClaim per chunk, and the first
            // UNITS / kClaim askers (eight) get kClaim units each.  The add for chunk r is issued before the
            // wave reports chunk r - 1 as done, and LDS operations of a wave execute in order: once
            // every wave is done with r - 1, all adds for r have been applied, so a fast wave's add
            // for r + 2 (same counter) cannot get in between.
            constexpr unsigned kClaim = S::UNITS / 8;
            auto help_stage = [&](int rel, bool report_done) {
                const int p = rel & 1;
                unsigned got = 0;
                if (fresh_lane() == 0) {
                    got = __hip_atomic_fetch_add(&tickets[p], kClaim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (report_done)                                   // chunk rel - 1 used the other buffer
                        __hip_atomic_fetch_add(&done[p ^ 1], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
                const unsigned unit0 = __builtin_amdgcn_readfirstlane(got) - unsigned(rel >> 1) * (NW * kClaim);
                if (unit0 < unsigned(S::UNITS)) {
                    wait_ge(&done[p], unsigned(rel >> 1) * NW);        // chunk rel - 2 is finished: the buffer is free
                    for (unsigned u = 0; u < kClaim; ++u)
                        stage_direct((c_begin + rel) * CH, lds + p * BUF_FLOATS, int(unit0 + u));
                    __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0): the data is in LDS
                    if (fresh_lane() == 0)
                        __hip_atomic_fetch_add(&staged[p], kClaim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            };

            {
                float4 rec_w;
                fetch_records(c_begin, k0, k_cnt, rec_m, rec_w);       // on the way while chunk 0 is staged
                help_stage(0, false);
                if (lane < BATCH) *reinterpret_cast<float4 *>(wlds + lane * 4) = rec_w;
            }
            for (int rel = 0; rel < n_rel; ++rel) {
                const bool more = rel + 1 < n_rel;
                uint32_t nk0 = 0, nk_cnt = 0, nrec_m = 0;
                float4 nrec_w = make_float4(0.f, 0.f, 0.f, 0.f);
                if (more) fetch_records(c_begin + rel + 1, nk0, nk_cnt, nrec_m, nrec_w);   // lands during the records below
                wait_ge(&staged[rel & 1], unsigned((rel >> 1) + 1) * S::UNITS);
                compute(rel, k0, k_cnt, rec_m);
                // every LDS read of this chunk has returned (the record loop waits for its loads)
                if (more) {
                    { const int lw = fresh_lane(); if (lw < BATCH) *reinterpret_cast<float4 *>(wlds + lw * 4) = nrec_w; }
                    k0 = nk0; k_cnt = nk_cnt; rec_m = nrec_m;
                    help_stage(rel + 1, true);
                }
            }
        } else {
            // ---- register staging path: fixed assignment, one barrier per chunk ----
            {
                float4 rec_w;
                stage(0);
                fetch_records(c_begin, k0, k_cnt, rec_m, rec_w);
                if (lane < BATCH) *reinterpret_cast<float4 *>(wlds + lane * 4) = rec_w;
                __syncthreads();
            }
            for (int rel = 0; rel < n_rel; ++rel) {
                // The next chunk goes to the other LDS buffer, which every wave has finished reading
                // (they all passed the barrier at the end of the previous iteration).
                const bool more = rel + 1 < n_rel;
                uint32_t nk0 = 0, nk_cnt = 0, nrec_m = 0;
                float4 nrec_w = make_float4(0.f, 0.f, 0.f, 0.f);
                if (more) {
                    stage(rel + 1);
                    fetch_records(c_begin + rel + 1, nk0, nk_cnt, nrec_m, nrec_w);
                }
                compute(rel, k0, k_cnt, rec_m);
                if (more) {
                    { const int lw = fresh_lane(); if (lw < BATCH) *reinterpret_cast<float4 *>(wlds + lw * 4) = nrec_w; }
                    k0 = nk0; k_cnt = nk_cnt; rec_m = nrec_m;
                    __syncthreads();
                }
            }
        }

        // ---- the partial sums of waves that had different channels are added through LDS ----
        if constexpr (PRIV) {
            // Waves on their own: two slots at a time go to LDS from every wave that had channels, and
            // wave s adds up slot s, in order of the waves, and writes its outputs.  (As a tree over the
            // waves, with one of them writing everything, it was slower.)
            const int parts = min(NW, a.c_in);
            v4f *red = reinterpret_cast<v4f *>(lds);
#pragma unroll
            for (int pass = 0; pass < FB / 2; ++pass) {
                __syncthreads();                         // the staging slots, or the pass before, are done with
                if (wave < parts) {
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int qd = 0; qd < 4; ++qd) {
                            const v16f &c = acc[2 * pass + u];
                            red[((wave * 2 + u) * 4 + qd) * 64 + lane] = v4f{c[4 * qd], c[4 * qd + 1], c[4 * qd + 2], c[4 * qd + 3]};
                        }
                }
                __syncthreads();
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    if (wave == 2 * pass + u) {
                        v4f sum[4];
#pragma unroll
                        for (int qd = 0; qd < 4; ++qd) sum[qd] = red[(u * 4 + qd) * 64 + lane];
#pragma unroll 3
                        for (int w = 1; w < parts; ++w)
#pragma unroll
                            for (int qd = 0; qd < 4; ++qd) sum[qd] += red[((w * 2 + u) * 4 + qd) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[2 * pass + u][e] = sum[e >> 2][e & 3];
                    }
            }
        } else if (ks_log2 > 0) {
            // channel splits of a chunk: split 2s+1 into 2s, then 2 into 0
            __syncthreads();                             // the staging buffers are free now
            float4 *red = reinterpret_cast<float4 *>(lds);
            for (int step = (1 << ks_log2) >> 1; step >= 1; step >>= 1) {
                const bool sender = ksplit >= step && ksplit < 2 * step;
                const bool receiver = ksplit < step;
                // slot of (filter block fbw, split): 16 float4 per lane
                const int fbw = wave - ksplit * fw;
                const int slot = ((sender ? ksplit - step : ksplit) * fw + fbw) * (16 * 64);
                if (sender) {
#pragma unroll
                    for (int s = 0; s < FB; ++s)
#pragma unroll
                        for (int qd = 0; qd < 4; ++qd)
                            red[slot + (s * 4 + qd) * 64 + lane] =
                                make_float4(acc[s][4 * qd], acc[s][4 * qd + 1], acc[s][4 * qd + 2], acc[s][4 * qd + 3]);
                }
                __syncthreads();
                if (receiver) {
#pragma unroll
                    for (int s = 0; s < FB; ++s)
#pragma unroll
                        for (int qd = 0; qd < 4; ++qd) {
                            const float4 p = red[slot + (s * 4 + qd) * 64 + lane];
                            acc[s][4 * qd] += p.x; acc[s][4 * qd + 1] += p.y; acc[s][4 * qd + 2] += p.z; acc[s][4 * qd + 3] += p.w;
                        }
                }
                __syncthreads();
            }
        }

        // ---- epilogue ----
        // Whole unit, or its last chunks: bias, ReLU, store (filters go back to their original
        // index).  A piece that takes over first adds what the previous workgroup left in the
        // output tensor; a piece that hands on stores the raw sums there instead.
        // the patch coordinates are recomputed here instead of being kept in registers across the loop
        int pidx_e = tile * 64 + lane;
        asm volatile("" : "+v"(pidx_e));
        const bool writer = active && (PRIV ? wave < FB : ksplit == 0) && pidx_e < a.n_patches;
        if constexpr (VEC && SPLIT) {
            if (takes_over) {
                // The predecessor (id - 8: same set, previous range) started before this workgroup
                // and ran the shared unit first, so this wait is normally over before it begins.
                // It is bounded all the same; if it ever expires the outputs are poisoned with NaN.
                // One wave polls, and only its successful read is followed by the (costly)
                // device-wide acquire; the barrier passes it on to the other waves.
                if (wave == 0) {
                    bool there = false;
                    for (int guard = 0; guard < (a.spin_limit >> 2) && !there; ++guard) {
                        there = __hip_atomic_load(a.flags + (blockIdx.x - set_stride), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.epoch;
                        if (!there) __builtin_amdgcn_s_sleep(8);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    if (!there && lane == 0) {
                        sync_words[6] = 1u;
                        __hip_atomic_store(a.err, kErrHandOverWait, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                    }
                }
                __syncthreads();
                // Add what the predecessor left in the output tensor: generated assembly, all loads of
                // two slots in flight at once (the workgroups that share a unit wait for one another
                // here, one after the other, so this is on the critical path of the layer).  A lane
                // without a patch, a row below the image and an empty slot read nothing or something
                // that is never stored.
                {
                    const int lt = fresh_lane();
                    const int pidx_t = tile * 64 + lt;
                    const bool pv = pidx_t < a.n_patches;
                    const int n_t = pv ? pidx_t / per_img : 0, prem_t = pv ? pidx_t - n_t * per_img : 0;
                    const int ye_t = (prem_t / a.px) * 4, xe_t = min((prem_t % a.px) * 4, a.w - 4);
                    uint32_t voff[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        voff[i] = (pv && ye_t + i < a.h) ? uint32_t(((n_t * a.c_out * a.h + ye_t + i) * a.w) + xe_t) * 4u : kOutOfRange;
                    uint32_t so[FB];
#pragma unroll
                    for (int s = 0; s < FB; ++s) {
                        const int f = __builtin_amdgcn_readfirstlane(__float_as_int(out_tab[2 * s]));
                        so[s] = uint32_t(max(f, 0)) * uint32_t(hw) * 4u;
                    }
                    v4u yrsrc;
                    {
                        const uint64_t ya = reinterpret_cast<uint64_t>(a.y);
                        yrsrc.x = __builtin_amdgcn_readfirstlane(uint32_t(ya));
                        yrsrc.y = __builtin_amdgcn_readfirstlane(uint32_t(ya >> 32) & 0xFFFFu);
                        yrsrc.z = __builtin_amdgcn_readfirstlane(a.y_bytes);
                        yrsrc.w = 0x00020000u;
                    }
                    asm volatile(
#include "pconv_tiled_takeover.inc"
                        : "+{v[64:79]}"(acc[0]), "+{v[80:95]}"(acc[1]), "+{v[96:111]}"(acc[2]), "+{v[112:127]}"(acc[3])
                        : [voff0] "v"(voff[0]), [voff1] "v"(voff[1]), [voff2] "v"(voff[2]), [voff3] "v"(voff[3]),
                          [rsrc] "s"(yrsrc), [so0] "s"(so[0]), [so1] "s"(so[1]), [so2] "s"(so[2]), [so3] "s"(so[3])
                        : "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35",
                          "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47",
                          "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "memory");
                }
            }
        }
        if constexpr (VEC) {
            // a wait of this workgroup ran out: its sums cannot be trusted
            if (__hip_atomic_load(&sync_words[6], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
#pragma unroll
                for (int s = 0; s < FB; ++s) acc[s] = __builtin_nanf("");
            }
        }
        if (writer) {
            const int n_e = pidx_e / per_img, prem_e = pidx_e - n_e * per_img;
            const int ye = (prem_e / a.px) * 4;
            const int xe = VEC ? min((prem_e % a.px) * 4, a.w - 4) : (prem_e % a.px) * 4;
            const int ho = a.h, wo = a.w;
#pragma unroll
            for (int s = 0; s < FB; ++s) {
                if (PRIV && s != wave) continue;
                const int f = __float_as_int(out_tab[2 * s]);
                if (f < 0) continue;
                const float b = hands_on ? 0.0f : out_tab[2 * s + 1];
                if constexpr (VEC) {
                    if (a.pool) {
                        // 2x2 / stride-2 max-pool of the lane's 4x4 outputs (the patch is aligned to the
                        // pooling grid: rows at multiples of 4, columns at a multiple of 4 or at W - 4
                        // with W even): two rows of two pooled values.  Bias and ReLU first.
                        const int hp = ho >> 1, wp = wo >> 1;
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            if ((ye >> 1) + i >= hp) continue;
                            float m[2];
#pragma unroll
                            for (int k = 0; k < 2; ++k) {
                                float v = fmaxf(fmaxf(acc[s][(2 * i) * 4 + 2 * k], acc[s][(2 * i) * 4 + 2 * k + 1]),
                                                fmaxf(acc[s][(2 * i + 1) * 4 + 2 * k], acc[s][(2 * i + 1) * 4 + 2 * k + 1])) + b;
                                m[k] = a.relu ? fmaxf(v, 0.0f) : v;
                            }
                            float *dst = reinterpret_cast<float *>(y) + ((size_t(n_e) * a.c_out + f) * hp + (ye >> 1) + i) * wp + (xe >> 1);
                            *reinterpret_cast<float2 *>(dst) = make_float2(m[0], m[1]);
                        }
                        continue;
                    }
                    if (a.sub2) {
                        // stride 2: of the lane's 4x4 outputs the two even rows, and of each the two even
                        // columns (the patch starts at a multiple of 4, or at W - 4 in the last patch of a row)
                        const int h2 = (ho + 1) >> 1, w2 = (wo + 1) >> 1, k0 = xe & 1;
#pragma unroll
                        for (int i = 0; i < 4; i += 2) {
                            if (ye + i >= ho) continue;
                            float o[2];
#pragma unroll
                            for (int kk = 0; kk < 2; ++kk) {
                                float v = (k0 ? acc[s][i * 4 + 2 * kk + 1] : acc[s][i * 4 + 2 * kk]) + b;
                                o[kk] = a.relu ? fmaxf(v, 0.0f) : v;
                            }
                            float *dst = reinterpret_cast<float *>(y) + ((size_t(n_e) * a.c_out + f) * h2 + ((ye + i) >> 1)) * w2 + ((xe + k0) >> 1);
                            dst[0] = o[0];
                            if (((xe + k0) >> 1) + 1 < w2) dst[1] = o[1];
                        }
                        continue;
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (ye + i >= ho) continue;
                        float *dst = reinterpret_cast<float *>(y) + ((size_t(n_e) * a.c_out + f) * ho + ye + i) * wo + xe;
                        float o[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) o[k] = acc[s][i * 4 + k];
                        if (!hands_on) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) { o[k] += b; if (a.relu) o[k] = fmaxf(o[k], 0.0f); }
                        }
                        *reinterpret_cast<float4 *>(dst) = make_float4(o[0], o[1], o[2], o[3]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int oy = ye + i;
                        if (oy >= ho || (a.sub2 && (oy & 1))) continue;
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            float v = acc[s][i * 4 + k] + b;
                            if (a.relu) v = fmaxf(v, 0.0f);
                            const int ox = xe + k;
                            if (ox >= wo) continue;
                            if (!a.sub2) st_act(y, act_at<T, LAYOUT>(n_e, f, oy, ox, a.c_out, ho, wo), v);
                            else if (!(ox & 1))
                                st_act(y, act_at<T, LAYOUT>(n_e, f, oy >> 1, ox >> 1, a.c_out, (ho + 1) >> 1, (wo + 1) >> 1), v);
                        }
                    }
                }
            }
        }
        if constexpr (VEC && SPLIT) {
            if (hands_on) {
                // the barrier orders every thread's stores before the release below, which makes
                // them visible to the whole device before the successor is told
                __syncthreads();
                if (threadIdx.x == 0)
                    __hip_atomic_store(a.flags + blockIdx.x, a.epoch, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <typename T, int LAYOUT, bool VEC, int NW, int CH, bool SPLIT, bool PRIV = false, bool SUB2 = false>
hipError_t launch_shape(const TiledArgs &a, int64_t wgs, hipStream_t st, int dev)
{
    // The kernel needs more dynamic LDS than the default limit: raised once per device (the flag is
    // set to the same value by every thread that gets here first).
    static std::atomic<bool> attr_done[64];
    constexpr size_t lds_bytes = Shape<NW, CH>::LDS_BYTES;
    if (dev < 0 || dev >= 64 || !attr_done[dev].load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_tiled_kernel<T, LAYOUT, VEC, NW, CH, SPLIT, PRIV, SUB2>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, int(lds_bytes));
        if (e != hipSuccess) return e;
        if (dev >= 0 && dev < 64) attr_done[dev].store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL((conv_tiled_kernel<T, LAYOUT, VEC, NW, CH, SPLIT, PRIV, SUB2>), dim3(unsigned(wgs)), dim3(NW * 64), lds_bytes, st, a);
    return hipGetLastError();
}

template <int NW, int CH>
hipError_t launch_any(const TiledArgs &a, int64_t wgs, hipStream_t st, bool vec, int layout, int dtype, int dev)
{
    if constexpr (NW == 16)
        if (a.priv) {                                    // (channels last: pconv_lone.hip has every call of the kind with vec)
            return dtype == PCONV_F32 ? launch_shape<float, PCONV_NHWC, false, NW, CH, false, true>(a, wgs, st, dev)
                                      : launch_shape<bf16_t, PCONV_NHWC, false, NW, CH, false, true>(a, wgs, st, dev);
        }
    if constexpr (NW == 16)
        if (vec && a.sub2 && a.w % 2 == 0) return launch_shape<float, PCONV_NCHW, true, NW, CH, false, false, true>(a, wgs, st, dev);
    if (vec)
        return a.split_units ? launch_shape<float, PCONV_NCHW, true, NW, CH, true>(a, wgs, st, dev)
                             : launch_shape<float, PCONV_NCHW, true, NW, CH, false>(a, wgs, st, dev);
    if (dtype == PCONV_F32)
        return layout == PCONV_NCHW ? launch_shape<float, PCONV_NCHW, false, NW, CH, false>(a, wgs, st, dev)
                                    : launch_shape<float, PCONV_NHWC, false, NW, CH, false>(a, wgs, st, dev);
    return layout == PCONV_NCHW ? launch_shape<bf16_t, PCONV_NCHW, false, NW, CH, false>(a, wgs, st, dev)
                                : launch_shape<bf16_t, PCONV_NHWC, false, NW, CH, false>(a, wgs, st, dev);
}

// test overrides, see set_tiled_tuning / set_tiled_spin_limit
std::atomic<int> g_force_waves{0}, g_force_ks{-1}, g_force_split{-1};
constexpr double kShareGain = 0.97;
constexpr int kDefaultSpinLimit = 1 << 22;
std::atomic<int> g_spin_limit{kDefaultSpinLimit};

}  // namespace

void set_tiled_tuning(int waves, int ks_log2, int split_units)
{
    g_force_waves.store((waves == 8 || waves == 16) ? waves : 0);
    g_force_ks.store((ks_log2 >= 0 && ks_log2 <= 2) || (ks_log2 >= 4 && ks_log2 <= 7) ? ks_log2 : -1);
    g_force_split.store((split_units >= 0 && split_units <= 2) ? split_units : -1);
}

void set_tiled_spin_limit(int limit) { g_spin_limit.store(limit > 0 ? limit : kDefaultSpinLimit); }

bool tiled_supported(const pconv_handle *h, int n, int hin, int win, int stride, int layout, int dtype)
{
    (void)layout; (void)dtype;
    if (h->tiled.meta.size() >= kTiledMaxRecords || (stride != 1 && stride != 2)) return false;
    const int64_t patches = int64_t(n) * ((hin + 3) / 4) * ((win + 3) / 4);
    return patches < (int64_t(1) << 30);
}

bool tiled_preferred(int hin, int win, int stride)
{
    // Stride 2 stages four times the pixels it needs and, but for SUB2, forms four times the outputs it stores; without
    // SUB2 it was measured 1.6 to 3.4 times as fast as the gather kernel all the same (ResNet-50 shapes, batch 32,
    // inputs of 56x56, 28x28 and 14x14).  Smaller images are left to the gather kernel.
    return stride == 1 || int64_t(hin) * win >= 12 * 12;
}

// fp32 with channels last: the tensors laid out channels first before the convolution and back after it, or staged
// through registers in the layout they have.  The changes of layout take 4 us + 0.35 a MB of input, and 3 us + 0.36 a MB of
// output unless waves on their own store it (0.86 a MB); what they save grows with the chunks of channels, more so where
// pixels are no whole quads of channels, and with the output, which the other kernels store four bytes at a time.  us, with change
// and without: 128 channels @28, eight images 20, 34; 200 to 50 @112, 16 images 210, 802; 99 to 40 @56, one image 13, 119; but 8 to
// 16 @20, 20, 13.  With one line for all, 130 of 13 600 drawn layers that changed their layout took more than 1.1 times as long for it:
// - Quads of channels, 8 MB of input and more: 4 us + 0.35 a MB was too little for the smaller gains (76 to 13 @70, 39 images 69, 58,
//   72 to 8 @117, seven images 31, 26); 8 + 0.38 leaves 6 of 1 000 layers more than a tenth slower, for 26.
// - One chunk of channels stages in no more than the changes take unless the output is most of the call: with more than 1.5 MB of input, 18 MB
//   of output and three times the input leave 5 of 1 700, for 95 (4 to 5 @158x126, 44 images 59, 31; 5 to 13 @223x178, stride 2, four
//   images 19, 12; but 5 to 25 @209x212, 19 images 84, 151).
bool tiled_nchw_preferred(const pconv_handle *h, int n, int hin, int win, int stride)
{
    const bool pinned = g_force_waves.load() || g_force_ks.load() >= 0 || g_force_split.load() >= 0;
    const int64_t pixels_out = int64_t((hin - 1) / stride + 1) * ((win - 1) / stride + 1);
    const double x_mb = double(n) * h->c_in * hin * win * 4e-6;
    const double y_mb = double(n) * h->c_out * pixels_out * 4e-6;
    if (pinned || win < 4 || int64_t(n) * h->c_in * hin * win * 4 >= (int64_t(1) << 31) ||
        transpose_tiles(n, int64_t(hin) * win, h->c_in) > kTransposeMaxTiles || transpose_tiles(n, h->c_out, pixels_out) > kTransposeMaxTiles ||
        !tiled_supported(h, n, hin, win, stride, PCONV_NCHW, PCONV_F32) || !tiled_preferred(hin, win, stride))
        return false;
    const bool quads = h->c_in % 4 == 0;
    const bool many = h->c_in > 32 || (h->c_in > 16 && h->c_out > 8) || (!quads && h->c_in > 4) || (y_mb > 12.0 && y_mb > x_mb);
    const int chunks = (h->c_in + kTileCH - 1) / kTileCH;
    if (chunks == 1) return many && (x_mb < 1.5 || (y_mb > 18.0 && y_mb > 3.0 * x_mb));
    return many && (x_mb < 8.0 || (quads ? 8.0 + 0.38 * x_mb < 1.13 * chunks + 1.4 * y_mb : 4.0 + 0.35 * x_mb < 4.88 * chunks + 1.4 * y_mb));
}

bool tiled_pool_supported(const pconv_handle *h, int n, int hin, int win, int layout, int dtype)
{
    return tiled_supported(h, n, hin, win, 1, layout, dtype) && dtype == PCONV_F32 && layout == PCONV_NCHW &&
           win >= 4 && win % 2 == 0 && hin >= 2 && int64_t(n) * h->c_in * hin * win * 4 < (int64_t(1) << 31);
}

namespace {

__global__ void fill_words_kernel(uint32_t *p, int count, uint32_t value)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = value;
}

// Device address of `scratch` on the handle's device (which is the current one), looked up on the
// first call per device and kept; nullptr (message set) if the runtime refuses.
uint32_t *static_flags(int dev)
{
    static std::atomic<uint32_t *> ptrs[64];
    if (dev < 0 || dev >= 64) { set_error("pconv_conv2d_static: device index out of range"); return nullptr; }
    uint32_t *p = ptrs[dev].load(std::memory_order_acquire);
    if (p) return p;
    void *sym = nullptr;
    const hipError_t e = hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !sym) {
        set_error(std::string("pconv_conv2d_static: hipGetSymbolAddress: ") + hipGetErrorName(e));
        return nullptr;
    }
    p = static_cast<uint32_t *>(sym);
    ptrs[dev].store(p, std::memory_order_release);   // (every thread gets the same address)
    return p;
}

std::atomic<uint32_t> g_static_calls{0};             // epochs of the calls that use `scratch`

bool is_capturing(hipStream_t st)
{
    if (!st) return false;                               // (the default stream cannot be captured)
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    return hipStreamIsCapturing(st, &status) != hipSuccess || status != hipStreamCaptureStatusNone;
}

}  // namespace

namespace {

// How a call is spread over the chip.
struct TiledPlan {
    int nw;               // waves per workgroup
    bool vec, split, one_set, priv, halves;
    int lone_waves;       // priv with vec: waves of a workgroup, 16, 8 or 4
    int ks_log2;
    int tail_tiles;       // tiles at the end that a second launch computes, by waves on their own
};

TiledPlan plan_tiled(const pconv_handle *h, int n, int hin, int win, int layout, int dtype, bool pool, bool sub2,
                     bool may_share = true)
{
    TiledPlan p{};
    p.lone_waves = 16;
    const int64_t x_bytes = int64_t(n) * h->c_in * hin * win * 4, y_bytes = int64_t(n) * h->c_out * hin * win * 4;
    const int force_waves = g_force_waves.load(), force_ks = g_force_ks.load(), force_split = g_force_split.load();
    p.vec = dtype == PCONV_F32 && layout == PCONV_NCHW && win >= 4 && x_bytes < (int64_t(1) << 31);
    // Shape: 16-wave workgroups, one per compute unit.  A layer whose input channels fit one 4-channel
    // chunk is all staging and output stores: there two 8-wave workgroups per compute unit overlap
    // one's stores with the other's loads.
    p.nw = force_waves ? force_waves : (h->c_in <= 4 ? 8 : 16);
    const int ch = p.nw == 16 ? 8 : 4;
    const int n_chunks = (h->c_in + ch - 1) / ch, px = (win + 3) / 4;
    const int64_t patches = int64_t(n) * ((hin + 3) / 4) * px;
    const int n_tiles = int((patches + 63) / 64);
    const int cus = h->cus > 0 ? h->cus : 256;
    const int slots = cus * (16 / p.nw);                 // workgroups that can run at once
    const int blocks = h->tiled.num_blocks;
    // Sharing a unit between workgroups needs fp32 outputs written 128 bits at a time, the full-size
    // output tensor for the partial sums (no fused max-pool, no stride 2), below 2 GiB (they are read
    // back with range-checked buffer loads), and tiles whose borders fall between patch rows: where the
    // image width is no multiple of 4 the last patch of a row overlaps its neighbour, and both
    // write the columns they share; if the two lay in different tiles, their workgroups would read
    // and overwrite each other's partial sums.
    const bool rows_whole = win % 4 == 0 || n_tiles == 1 || 64 % px == 0;
    const bool can_split = may_share && p.vec && !pool && !sub2 && y_bytes < (int64_t(1) << 31) && rows_whole;
    // waves on their own: rows of patches by 128-bit loads, or channels last in whole quads
    const bool can_priv = p.nw == 16 && (p.vec || (layout == PCONV_NHWC && h->c_in % 4 == 0));
    const int64_t whole_units = int64_t(n_tiles) * ((blocks + p.nw - 1) / p.nw);
    auto units_of = [&](int ks) { return (blocks + (p.nw >> ks) - 1) / (p.nw >> ks); };   // filter groups per tile
    const double records = double(h->tiled.meta.size()) * p.nw / blocks / n_chunks;       // of a whole unit's chunk
    const double visits = double(h->tiled.visits) / blocks, recs = double(h->tiled.meta.size()) / blocks;
    // Whole units with stride 2 are priced as with stride 1, although with even widths they do a quarter of the FMAs: staging
    // is what such a unit takes its time for.
    // Waves on their own.  fp32 NCHW (pconv_lone.hip), 16, 8 or 4 waves per workgroup, so that a compute unit holds one, two
    // or four: tiles x groups workgroups of v visited channels and r records.  A round is a start and an end and the work of
    // the workgroups of a compute unit, which takes longer per workgroup where fewer than four waves share a SIMD.
    // Fitted to 62 layers with 1 to 64 images (5 % off on average; 256 channels @56, one image 18 us with 16, 22, 32;
    // 64 @224, one image 33, 23, 19; 512 @14, 32 images 113, 105, 100); a sixth more where tiles cut rows of patches.
    // Two slots a workgroup (the fourth row, 16 waves): one pass of sums for two, a round costs 3.1 for 4.7.  Fitted to 6 600
    // drawn layers (9 % off).  Priced with the first row, 1 130 of 7 400 layers with few units took 4 or 8 waves and 1.1 to 1.4
    // times as long: 11 to 44 channels @12x14, 27 images 6.7 us for 4.9, 24 to 329 @19, two images 6.1 for 4.8.
    // Every workgroup of a tile reads the same channels.  They come from the L2 while the tiles that the 32 compute units of an
    // XCD work on at a time (4 KB a channel) fit its 4 MB: up to 25 TB/s were seen then, 16 with 6 to 9 MB, 13 with more; so what does
    // not fit is charged at 33 TB/s on top.  Priced without, 491 to 63 filters @79x82, stride 2, 36 images took 603 us for the
    // 254 of whole units, 412 to 57 @120x144, seven images 301 for 153.
    // Channels last 3.3 for 16 channels (128 @28, eight images: 38 us, whole units 120, 81, 62).
    struct LoneCost { double base, round, visit, record, work[4]; };
    static constexpr LoneCost kLoneCost[4] = {{1.84, 4.70, 0.0437, 0.0113, {1.0}}, {2.65, 3.40, 0.0395, 0.0151, {1.24, 2.0}},
                                              {1.93, 3.46, 0.0382, 0.0153, {2.27, 2.81, 3.52, 4.0}}, {1.1, 3.1, 0.053, 0.017, {1.0}}};
    auto lone_time = [&](int waves, bool halves, const LoneTiles &t, double v, double r) {
        const LoneCost &c = kLoneCost[halves ? 3 : waves == 16 ? 0 : waves == 8 ? 1 : 2];
        const int most = 16 / waves, groups = halves ? 2 * blocks : blocks;
        const bool quarter = sub2 && win % 2 == 0;
        const double units = double(t.tiles) * groups, n = std::ceil(units / cus), full = std::floor(n / most);
        const double work = (c.visit * v + c.record * r) * (t.cut ? 1.17 : 1.0) * (quarter ? 0.7 : 1.0);
        const int left = int(n - full * most);
        const double in_flight = std::min(double(t.tiles) / 8, std::max(1.0, cus / 8.0 * most / groups)), mb = in_flight * h->c_in * 4e-3;
        const double mb_read = units * v * (quarter ? 5 : 6) * 1024e-6 * t.lanes / 64;
        return c.base + full * (c.round + most * work) + (left > 0 ? c.round + c.work[left - 1] * work : 0.0) + (mb > 4.0 ? mb_read * (1.0 - 4.0 / mb) / 33.0 : 0.0);
    };
    // the number of waves with the smallest estimate
    auto lone_best = [&](const LoneTiles &t, int &waves) {
        double best = 0.0;
        for (int w = 16; w >= 4; w /= 2) {
            const double time = lone_time(w, false, t, visits, recs);
            if (w == 16 || time < best) { best = time; waves = w; }
        }
        return best;
    };
    const double lone_last = 10.0 + 3.3 * ((h->c_in + 15) / 16);     // (channels last: a round)
    if (whole_units > slots / 2) {
        if (can_split && p.nw == 16) {
            // Many units, but not a multiple of the number of compute units: whole units leave part of
            // the chip idle in the last round.  Dealing the chunks of all units evenly (every workgroup
            // one contiguous share, over all workgroups as one set) costs each workgroup further start-ups
            // and the partial sums through memory with a device-wide release and acquire, taken as ten
            // chunks; a last round with few units runs faster than a full one (measured: 0.87 of it at
            // 53 % busy).  So it pays for few, long units only (512 channels @28, 64 images, 392 units of 64
            // chunks).  With seven chunks 40 layers whose form that changes took 1.13 times as long on
            // average: 256 channels @56, 32 images 290 -> 269 us and 138 -> 394 @28, 55 images 234 -> 181, but
            // 128 @112, 32 images 286 -> 331, and 256 -> 8 @82x112, 17 images 32 -> 80, whose second launch
            // and waves on their own (below) sharing rules out.
            constexpr double kShareOverhead = 10.0;
            const double full = double(whole_units / slots), rest = double(whole_units % slots) / slots;
            const double t_whole = n_chunks * (full + (rest > 0.0 ? 0.72 + 0.28 * rest : 0.0));
            const double t_share = double(whole_units) * n_chunks / slots + kShareOverhead;
            if (t_share < kShareGain * t_whole) p.split = p.one_set = true;
        }
        if (p.vec && can_priv && !p.split && force_split < 0 && force_ks < 0) {
            const double full = double(whole_units / slots), rest = double(whole_units % slots) / slots;
            const double round = 6.0 + n_chunks * (2.0 + 1.9 * records / 142.0), last = rest > 0.0 ? (0.72 + 0.28 * rest) * round : 0.0;
            double t_best = full * round + last;
            // A last round with few units: their tiles go to a second launch, in which the waves work on their
            // own and which takes a fraction of a round (128 channels @112, 32 images: 784 units are 3.06
            // rounds, 323 us; 280 with the tiles of the last 16 units apart).
            const int main_tiles = int(int64_t(full) * (slots / 8) / units_of(0)) * 8, tail = n_tiles - main_tiles;
            if (full > 0.0 && rest > 0.0 && main_tiles > 0) {
                const LoneTiles t = lone_tiles(patches, px, lone_base(int64_t(main_tiles) * 64, px), blocks, slots);
                int waves = 16;
                const double t_tail = 0.5 + lone_best(t, waves);
                if (t_tail < 0.8 * last) { p.tail_tiles = tail; p.lone_waves = waves; t_best = full * round + t_tail; }
            }
            // Up to three blocks of filters leave most of a whole unit's waves idle: waves on their own may still be
            // faster (160 to 8 channels @95x102, 44 images: 81 us for 117).  Four to seven blocks are asked neither here nor
            // below and stay whole units, also where waves on their own are faster: 64 to 16 @112x138, stride 2, 32 images 46 us,
            // 32 with 4 waves; 128 to 16 @112, 16 images 51, 31; but 128 to 28 54, 51.  Nor are they asked where units are shared.
            if (blocks < p.nw / 4) {
                const LoneTiles t = lone_tiles(patches, px, 0, blocks, slots);
                int waves = 16;
                if (lone_best(t, waves) < 0.9 * t_best) {
                    p.priv = true; p.ks_log2 = 4; p.tail_tiles = 0; p.lone_waves = waves;
                }
            }
        }
        // Waves on their own, two or four workgroups to a compute unit, have no last round to speak of (512 channels
        // @28, 64 images, 12 uneven patterns: 436 us as whole units, 380 as shared ones, 365 with 4 waves).  The estimates above
        // are what a unit takes by itself; with the chip full and its waves busy it is 1.37 times that, taken as 1.25 so that fewer
        // layers lose by the change (of 1 500 drawn ones five take more than 1.1 times what the units take), shared units 1.28;
        // even widths with stride 2, which form a quarter of the FMAs, 1.05.  Waves without a block of filters leave the others
        // their share of the record loop: priced as busy, 8 to 12 blocks took up to 1.4 times the time of whole units (10 to 75 filters
        // @134x160, 41 images 118 us for 101, 32 to 35 @204x207, 37 images 178 for 143), and so did stride 2 (200 to 460 @64, eight images
        // 127 for 103).  With the pool 1.1, as the outputs stored are a quarter (10 to 144 @172x206, five images 32.6 for 25.9).
        if (p.vec && can_priv && blocks >= p.nw / 2 && force_split < 0 && force_ks < 0) {
            const double busy = double(blocks) / (units_of(0) * p.nw);
            const double chunk = 2.0 + 1.9 * records * busy / 142.0, full = double(whole_units / slots), rest = double(whole_units % slots) / slots;
            const double t_units = p.split ? 1.28 * chunk * (double(whole_units) * n_chunks / slots + 10.0)
                                           : (sub2 && win % 2 == 0 ? 1.05 : pool ? 1.1 : 1.25) * (6.0 + n_chunks * chunk) * (full + (rest > 0.0 ? 0.72 + 0.28 * rest : 0.0));
            const LoneTiles t = lone_tiles(patches, px, 0, blocks, slots);
            int waves = 16;
            if (lone_best(t, waves) < 0.97 * t_units && p.tail_tiles == 0) {
                p.priv = true; p.ks_log2 = 4; p.split = p.one_set = false; p.lone_waves = waves;
            }
        }
    } else {
        // Few units: the form with the smallest estimate, in microseconds, fitted to the VGG-16 layers
        // with one and four images.
        double best = 0.0;
        auto consider = [&](double t, bool split, int ks, bool priv, bool halves = false, int waves = 16) {
            if (best == 0.0 || t < best) { best = t; p.split = split; p.ks_log2 = ks; p.priv = priv; p.halves = halves; p.lone_waves = waves; }
        };
        // whole units, the waves of a workgroup splitting the channels of a chunk 1, 2 or 4 ways: a chunk
        // costs about 2 for its staging and 1.9 for 142 records on the whole workgroup (256 channels
        // @56: 133, 98, 84 us; register staging, which nothing overlaps, 2.4 and 4.8 in quads of
        // channels, 8 and 4 otherwise, all with few units: a full chip stages slower, see
        // stage_quads); an eighth of the tiles shares the compute units of one XCD
        // (`full`: more than a quarter of the chip's workgroups of 16 waves: they start together, and the memory shows;
        // priced as alone, 8 to 512 channels @80 with stride 2, two images took 13.7 us for the 9.1 of waves on their own,
        // 16 to 128 @112, three images 17.0 for 14.6, 32 to 256 @56, eight images 23.8 for 20.1; with 8 waves, 3 channels
        // @224, one image, the channels split two ways in 196 workgroups are still faster than 98 whole units, 12.1 for 13.6; with the
        // pool, which stores a quarter, 7: priced as without, 5 to 429 @118x140, one image 13.2 for 10.7, 16 to 118 @175 17.8 for 14.5)
        const bool quads = layout == PCONV_NHWC && h->c_in % 4 == 0;
        const double t_stage = p.vec ? 2.0 : quads ? 2.4 : 8.0, t_records = p.vec ? 1.9 : quads ? 4.8 : 4.0;
        const double chunk_scale = p.nw == 16 ? 1.0 : 0.5;
        for (int ks = 0; ks <= 2; ++ks) {
            if (ks > 0 && int64_t(n_tiles) * units_of(ks - 1) > slots / 2) break;
            const double rounds = std::ceil(double((n_tiles + 7) / 8) * units_of(ks) / (slots / 8.0));
            const bool full = p.vec && p.nw == 16 && int64_t(n_tiles) * units_of(ks) > slots / 4;
            consider(rounds * ((full ? pool ? 7.0 : 10.0 : 6.0) + (full ? 1.08 : 1.0) * chunk_scale * n_chunks * (t_stage + t_records * records / 142.0 / (1 << ks))), false, ks, false);
        }
        // units shared by P workgroups, which pass the sums on one after the other (256 channels @56, one
        // image: 99 us, four: 83; 192 to 128 @56, 12 images 106, waves on their own 85)
        if (can_split)
            consider(1.45 * (6.0 + 4.6 * chunk_scale * whole_units * n_chunks / slots + std::min(90.0, 10.0 * slots / double(whole_units))), true, 0, false);
        // one filter block per workgroup, every wave its own channels
        if (can_priv) {
            const LoneTiles t = lone_tiles(patches, px, 0, blocks, slots);
            const LoneTiles t2 = lone_tiles(patches, px, 0, 2 * blocks, slots);
            if (p.vec) {
                int waves = 16;
                const double t_all = lone_best(t, waves);
                consider(t_all, false, 4, true, false, waves);
                // two of the block's four filters per workgroup, where there are not enough blocks for the chip
                consider(lone_time(16, true, t2, double(h->tiled.half_visits) / (2 * blocks), recs / 2), false, 4, true, true);
            } else {
                consider(std::ceil(double(n_tiles) * blocks / slots) * lone_last, false, 4, true);
            }
        }
    }
    if (force_split >= 0) { p.split = can_split && force_split != 0; p.one_set = p.split && force_split == 2; if (p.split) { p.ks_log2 = 0; p.priv = false; } }
    if (force_ks >= 0) {
        p.priv = force_ks >= 4 && can_priv;
        p.halves = force_ks == 5 && p.priv;
        p.lone_waves = force_ks == 6 ? 8 : force_ks == 7 ? 4 : 16;
        p.ks_log2 = p.priv ? 4 : force_ks < 4 ? force_ks : 0;
        if (p.priv) p.split = p.one_set = false;
    }
    if (p.split && force_ks < 0) p.ks_log2 = 0;
    return p;
}

// Channels last: waves on their own store that way themselves, four bytes at a time, up to 6 MB (0.86 us a MB for
// 3 us and 0.36 a MB); what the others have stored changes its layout.
bool may_store_last(const pconv_handle *h, int n, int hin, int win, int stride)
{
    const int64_t out_bytes = int64_t(n) * h->c_out * ((hin - 1) / stride + 1) * ((win - 1) / stride + 1) * 4;
    return out_bytes < 6000000 && !(stride == 2 && win % 2 == 0);
}
bool stores_last(const TiledPlan &p) { return p.vec && p.priv && p.lone_waves == 16; }

}  // namespace

bool tiled_stores_last(const pconv_handle *h, int n, int hin, int win, int stride)
{
    return may_store_last(h, n, hin, win, stride) && stores_last(plan_tiled(h, n, hin, win, PCONV_NCHW, PCONV_F32, false, stride == 2));
}

void describe_tiled_plan(const pconv_handle *h, int n, int hin, int win, int stride, int layout, bool pool, pconv_plan &out)
{
    const TiledPlan p = plan_tiled(h, n, hin, win, layout, h->wdtype, pool, stride == 2);
    const int lone_waves = p.vec && p.priv ? p.lone_waves : 16;
    out.waves = lone_waves == 16 ? p.nw : lone_waves;
    out.ks_log2 = p.priv && p.halves ? 5 : p.ks_log2;
    out.split_units = p.split ? (p.one_set ? 2 : 1) : 0;
    out.tail_tiles = p.tail_tiles;
    if (p.vec && (p.priv || p.tail_tiles > 0)) {
        const int px = (win + 3) / 4;
        const int64_t patches = int64_t(n) * ((hin + 3) / 4) * px, first = (patches + 63) / 64 * 64 - int64_t(p.tail_tiles) * 64;
        const LoneTiles t = lone_tiles(patches, px, p.priv ? 0 : lone_base(first, px), int64_t(h->tiled.num_blocks) << (p.priv && p.halves ? 1 : 0),
                                       h->cus > 0 ? h->cus : 256);
        out.lone_patches = t.lanes; out.lone_cut = t.cut;
    }
}

bool tiled_shares_units(const pconv_handle *h, int n, int hin, int win)
{
    // the automatic choice of launch_conv_tiled for an fp32 NCHW call with stride 1 and no fused pool
    const TiledPlan p = plan_tiled(h, n, hin, win, PCONV_NCHW, PCONV_F32, false, false);
    return p.split && !p.one_set;
}

int launch_conv_tiled(const pconv_handle *h, const void *x, void *y, const float *bias, int n,
                      int hin, int win, int stride, int layout, int dtype, int relu, int pool, void *stream,
                      bool static_scratch, float *y_last)
{
    TiledArgs a;
    a.sub2 = stride == 2;
    a.x = x; a.y = y; a.bias = bias;
    a.slot_filter = h->d_slot_filter; a.chan_ptr = h->d_chan_ptr; a.meta = h->d_meta;
    a.w4 = reinterpret_cast<const float4 *>(h->d_w4);
    a.n_img = n; a.c_in = h->c_in; a.row_len = h->tiled.row_len; a.h = hin; a.w = win; a.c_out = h->c_out;
    a.py = (hin + 3) / 4; a.px = (win + 3) / 4;
    a.n_patches = n * a.py * a.px;
    a.n_tiles = (a.n_patches + 63) / 64;
    a.n_blocks = h->tiled.num_blocks;
    a.relu = relu; a.pool = pool;
    a.x_bytes = uint32_t(std::min<int64_t>(int64_t(n) * h->c_in * hin * win * 4, 0x7FFFFFFF));
    a.y_bytes = uint32_t(std::min<int64_t>(int64_t(n) * h->c_out * hin * win * 4, 0x7FFFFFFF));
    a.err = h->h_err; a.spin_limit = g_spin_limit.load();
    TiledPlan plan = plan_tiled(h, n, hin, win, layout, dtype, pool != 0, stride == 2);
    // A captured launch keeps its arguments: a replay would find the hand-over words as the one before
    // left them, with the value that means "handed over".  (With the static words a kernel clears them,
    // in every replay.)
    if (plan.split && !static_scratch && is_capturing(static_cast<hipStream_t>(stream)))
        plan = plan_tiled(h, n, hin, win, layout, dtype, pool != 0, stride == 2, false);
    const bool last = y_last && stores_last(plan) && may_store_last(h, n, hin, win, stride);
    if (!y && !last) { set_error("pconv_conv2d_ws: launch choices were pinned while the call began"); return PCONV_UNSUPPORTED; }
    const int nw = plan.nw, ch = nw == 16 ? 8 : 4;
    const bool vec = plan.vec;
    const int slots = (h->cus > 0 ? h->cus : 256) * (16 / nw);
    a.n_chunks = (h->c_in + ch - 1) / ch;
    a.split_units = plan.split; a.one_set = plan.one_set; a.priv = plan.priv; a.ks_log2 = plan.ks_log2;
    a.n_records = uint32_t(h->tiled.meta.size()) - 3u;
    a.n_tiles -= plan.tail_tiles;
    const int fw = nw >> a.ks_log2;
    a.n_groups = (a.n_blocks + fw - 1) / fw;
    const int64_t units = int64_t(a.n_tiles) * a.n_groups;
    if (units > 0x3FFFFFFF) { set_error("pconv_conv2d: too many workgroups"); return PCONV_UNSUPPORTED; }
    a.n_units = int(units);
    int64_t wgs;
    a.flags = nullptr; a.epoch = 0;
    if (a.split_units) {
        // one workgroup per slot, but no fewer than two chunks each
        const int64_t iters = units * a.n_chunks;
        wgs = std::min<int64_t>(std::min<int>(slots, kFlagWords), std::max<int64_t>(8, iters / 2));
        if (static_scratch) {
            // the one row of the device's static array, cleared by a small kernel ahead of the
            // convolution on the same stream (calls that overlap on one device would race here)
            if (wgs > kFlagWords) { set_error("pconv_conv2d_static: more workgroups than hand-over words"); return PCONV_UNSUPPORTED; }
            uint32_t *row = static_flags(h->device);
            if (!row) return PCONV_HIP_ERROR;
            hipLaunchKernelGGL(fill_words_kernel, dim3((kFlagWords + 255) / 256), dim3(256), 0,
                               static_cast<hipStream_t>(stream), row, kFlagWords, 0u);
            if (hipGetLastError() != hipSuccess) { set_error("pconv_conv2d_static: clearing the hand-over words failed"); return PCONV_HIP_ERROR; }
            const uint32_t call = g_static_calls.fetch_add(1u);
            a.flags = row;
            a.epoch = call + 1u ? call + 1u : 1u;
        } else {
            const uint32_t call = h->calls.fetch_add(1u);
            a.flags = h->d_flags + size_t(call % kFlagSlots) * kFlagWords;
            a.epoch = call + 1u ? call + 1u : 1u;
        }
    } else {
        wgs = a.priv ? (units + 7) / 8 * 8 : int64_t((a.n_tiles + 7) / 8) * 8 * a.n_groups;   // one per unit of the largest set, in every set
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    auto lone = [&](bool halves, int waves, int64_t patch_base) {
        return launch_conv_lone(h, static_cast<const float *>(x), last ? y_last : static_cast<float *>(y), bias, n, hin, win, stride, relu,
                                pool, halves, waves, patch_base, last, stream);
    };
    hipError_t e = vec && plan.priv ? lone(plan.halves, plan.lone_waves, 0)
                   : nw == 16       ? launch_any<16, 8>(a, wgs, st, vec, layout, dtype, h->device)
                                    : launch_any<8, 4>(a, wgs, st, vec, layout, dtype, h->device);
    if (e == hipSuccess && plan.tail_tiles > 0) e = lone(false, plan.lone_waves, lone_base(int64_t(a.n_tiles) * 64, a.px));
    if (e != hipSuccess) {
        set_error(std::string("pconv_conv2d (tiled kernel): ") + hipGetErrorName(e));
        return PCONV_HIP_ERROR;
    }
    if (y_last && !last)
        return launch_transpose(static_cast<const float *>(y), y_last, n, h->c_out, ((hin - 1) / stride + 1) * ((win - 1) / stride + 1), stream);
    return PCONV_OK;
}

}  // namespace pconv
