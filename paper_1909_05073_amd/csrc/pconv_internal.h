// Internal declarations shared by the host packer, the kernels' launchers and the C ABI.
#pragma once

#include <atomic>
#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "pconv.h"

namespace pconv {

constexpr int kFlagSlots = 64, kFlagWords = 1024;
constexpr int kLoneWaves = 16;         // waves of a workgroup of pconv_lone.hip
// The register-tiled kernel keeps a record index in 24 bits: a longer stream stays off the device,
// and the layer runs on the other kernels.
constexpr size_t kTiledMaxRecords = size_t(1) << 24;

// Thread-local message for pconv_last_error().
void set_error(const std::string &msg);
const char *get_error();

// Result of the host-side analysis + reorder (paper: layer-wise information extraction and
// filter kernel reorder).  "Position" i means the i-th filter in the sorted order.
struct Canonical {
    std::vector<uint16_t> perm;      // [F]     filter at position i
    std::vector<uint32_t> row_ptr;   // [F+1]   first kernel of position i
    std::vector<uint16_t> pat_cnt;   // [F][P]  kernels per pattern at position i
    std::vector<uint16_t> cin;       // [K]     input channel of kernel k
    std::vector<uint8_t>  pat;       // [K]     pattern id of kernel k (derivable from pat_cnt)
    std::vector<uint32_t> val_ptr;   // [K+1]   first stored weight of kernel k
    std::vector<uint32_t> vals_bits; // [nnz]   fp32 bit patterns (bf16 handles: value << 16)
};

// Device-side stream of the register-tiled kernel.  Filters are dealt into blocks of kTileFB
// filters ("slots"); for every (block, input channel) the records of that channel are stored
// contiguously, ordered by slot.  A record is one code (sub-mask with a specialised inner
// loop) of one kernel, with up to four weights in ascending tap order.
struct TiledStream {
    int num_blocks = 0;                 // ceil(F / kTileFB)
    int row_len = 0;                    // entries per chan_ptr row: round_up(C, kTileCH) + 1
    std::vector<int32_t>  slot_filter;  // [num_blocks * kTileFB] original filter index or -1
    std::vector<uint32_t> chan_ptr;     // [num_blocks][row_len]
    int64_t visits = 0;                 // (block, channel) pairs with a record
    int64_t half_visits = 0;            // (block, half of its slots, channel) triples with a record
    std::vector<uint32_t> meta;         // [R+1] record words (see pconv_tiled_codes.h), one pad
    std::vector<float>    w4;           // [R+1][4]
};

// A call's launch shape of the flat matrix-core kernel, once chosen (see choose_flat).
struct FlatCall { int n = 0, h = 0, w = 0, stride = 0, layout = 0, index = 0, r = 0; int64_t plane = 0, lds = 0; };

}  // namespace pconv

struct pconv_handle {
    int c_out = 0, c_in = 0, np = 0, wdtype = 0, device = -1;
    uint16_t table[PCONV_MAX_PATTERNS] = {0};
    int64_t K = 0, nnz = 0, device_bytes = 0;
    pconv::Canonical canon;
    pconv::TiledStream tiled;
    // device copies (generic gather kernel)
    int32_t  *d_perm = nullptr;
    uint32_t *d_row_ptr = nullptr;
    uint32_t *d_kern = nullptr;      // [K] cin | mask << 16
    uint32_t *d_val_ptr = nullptr;   // [K]
    float    *d_vals = nullptr;      // [nnz] fp32 (bf16 weights widened exactly)
    // device copies (register-tiled kernel)
    int32_t  *d_slot_filter = nullptr;
    uint32_t *d_chan_ptr = nullptr;
    uint32_t *d_lone_bounds = nullptr, *d_lone_visits = nullptr;              // (one allocation; fp32 handles only)
    uint32_t *d_meta = nullptr;
    float    *d_w4 = nullptr;
    // device copies (matrix-core kernels, bf16 handles only): the masked weights as dense
    // [filter][channel] matrices per tap, in blocks of 32 filters and 16 channels, the nine taps of a
    // block next to each other: [fpad / 32][cb16 + 1][9][32][16] bf16, fpad = c_out rounded up to 32,
    // cb16 = c_in rounded up to 32, in sixteens (the last block of a row is zeros); and per (block of 32
    // channels, block of 32 filters) a word whose bit 2 * tap + half says whether that
    // (tap, 16 channels, 32 filters) block holds any kept weight
    uint16_t *d_wdense = nullptr;
    uint32_t *d_wnz = nullptr;
    int wd_full = 0;                 // 1: every such block that lies inside the layer holds a kept weight
    // Hand-over words of the tiled kernel: workgroups that share a unit of work signal each other
    // through kFlagWords words; every call takes the next of kFlagSlots such rows and a fresh
    // value, so calls that overlap on different streams do not see each other's signals.
    uint32_t *d_flags = nullptr;     // [kFlagSlots][kFlagWords], zero at start
    mutable std::atomic<uint32_t> calls{0};
    // Sticky error word of the kernels launched on this handle: pinned host memory that the device
    // writes (non-zero = a bounded wait inside a kernel ran out) and that the next call on the
    // handle reads without touching the device.
    uint32_t *h_err = nullptr;
    // launch shapes of the last few kinds of calls: the choice takes 1.3 us, a third of a call's launch
    mutable std::mutex flat_mutex;
    mutable pconv::FlatCall flat_calls[4];
    mutable unsigned flat_next = 0;
    int cus = 0;                     // compute units of `device`, read once at pack time
};

namespace pconv {

// Host analysis + reorder.  Returns PCONV_OK or an error status (message set).
int build_canonical(const float *w, const uint8_t *pid, const uint8_t *conn, const uint16_t *table,
                    int np, int c_out, int c_in, int wdtype, Canonical &out);

int project_weights(const float *w, const uint16_t *table, int np, int c_out, int c_in, int64_t keep,
                    uint8_t *pattern_id, uint8_t *conn);

// chan_mid: [num_blocks][c_in] first record of slots 2 and 3 of a channel (what build_lone_lists needs)
void build_tiled_stream(const Canonical &cn, const uint16_t *table, int np, int c_out, int c_in,
                        TiledStream &out, std::vector<uint32_t> &chan_mid);

// The lists that pconv_lone.hip walks: the first visit of each wave, [num_blocks][all slots, slots 0 and 1, slots 2
// and 3][kLoneWaves + 1], and behind them {first record, channel | records << 16} of every visited channel.
inline size_t lone_bounds_words(const TiledStream &ts) { return size_t(ts.num_blocks) * 3 * (kLoneWaves + 1); }
std::vector<uint32_t> build_lone_lists(const TiledStream &ts, const std::vector<uint32_t> &chan_mid, int c_in);

// Kernel launchers (pconv_kernels.hip, pconv_tiled.hip).  All return a pconv_status.
int launch_conv_generic(const pconv_handle *h, const void *x, void *y, const float *bias, int n,
                        int hin, int win, int stride, int layout, int dtype, int relu, void *stream);
// static_scratch: take the hand-over words from the code object's static array instead of the handle.  y_last: fp32
// NCHW calls only, not with pool: where the outputs go with channels last; y is work space, and null where tiled_stores_last.
int launch_conv_tiled(const pconv_handle *h, const void *x, void *y, const float *bias, int n,
                      int hin, int win, int stride, int layout, int dtype, int relu, int pool, void *stream,
                      bool static_scratch = false, float *y_last = nullptr);
// fp32 NCHW with few units of work: every wave on its own (pconv_lone.hip), from patch `patch_base` on.
struct LoneTiles { int lanes; bool cut; int64_t tiles; };        // patches of a tile, tiles that cut rows, their number
LoneTiles lone_tiles(int64_t patches, int px, int64_t patch_base, int64_t groups, int slots);
// Where a launch for the patches from `first` on begins: at a row of patches, if a tile can hold one (up to px - 1
// patches are computed twice).
inline int64_t lone_base(int64_t first, int px) { return px <= 64 ? first - first % px : first; }
hipError_t launch_conv_lone(const pconv_handle *h, const float *x, float *y, const float *bias, int n, int hin, int win,
                            int stride, int relu, int pool, bool halves, int waves, int64_t patch_base, bool last, void *stream);
// whether an fp32 call with channels last is better off with its tensors' layout changed before and after
bool tiled_nchw_preferred(const pconv_handle *h, int n, int hin, int win, int stride);
// whether the convolution of such a call stores its outputs with channels last itself, so that launch_conv_tiled needs no y
bool tiled_stores_last(const pconv_handle *h, int n, int hin, int win, int stride);
// whether the tiled kernel can write the 2x2 max-pooled output directly (pool = 1)
bool tiled_pool_supported(const pconv_handle *h, int n, int hin, int win, int layout, int dtype);
bool tiled_supported(const pconv_handle *h, int n, int hin, int win, int stride, int layout, int dtype);
// whether pconv_conv2d (fp32 NCHW, stride 1) would let workgroups share tiles of this call, which a
// fused max-pool rules out
bool tiled_shares_units(const pconv_handle *h, int n, int hin, int win);
// the launch choices of launch_conv_tiled for a call (fills all but `kernel`)
void describe_tiled_plan(const pconv_handle *h, int n, int hin, int win, int stride, int layout, bool pool, pconv_plan &out);
// plain vector-FMA rate of the device (see pconv_debug_measure_fma_peak)
int measure_fma_peak(double *tflops);
// whether the automatic policy should take the tiled kernel for a call it supports
bool tiled_preferred(int hin, int win, int stride);
// Test override of the tiled kernel's launch choices: waves per workgroup (8 or 16, anything else =
// automatic), log2 of the channel split inside a workgroup (0..2, 4 or 5, anything else = automatic), and
// whether workgroups may share a unit of work (0 / 1, anything else = automatic).
void set_tiled_tuning(int waves, int ks_log2, int split_units);
// Test override of the iteration limit of the kernels' bounded waits (<= 0 restores the default).
void set_tiled_spin_limit(int limit);
// bf16 layers on the matrix cores (pconv_mfma.hip)
bool mfma_supported(const pconv_handle *h, int dtype, int n, int hin, int win);
bool mfma_preferred(const pconv_handle *h);
int launch_conv_mfma(const pconv_handle *h, const void *x, void *y, const float *bias, int n,
                     int hin, int win, int stride, int layout, int relu, void *stream);
// The main matrix-core kernel (pconv_mfma_flat.hip); false (nothing launched) if it does not serve the call.
bool launch_conv_flat(const pconv_handle *h, const void *x, void *y, const float *bias, int n, int hin, int win,
                      int stride, int layout, int relu, void *stream, int &rc);
// index of the launch shape that kernel would take, -1 if it does not serve the call
int flat_shape_of(const pconv_handle *h, int n, int hin, int win, int stride, int layout);
// Test override of that choice (an index out of range restores the automatic one).
void set_flat_shape(int index);
// masked weights of a bf16 handle in the matrix-core kernel's layout (see pconv_handle::d_wdense)
void build_dense_taps(const Canonical &cn, const uint16_t *table, int c_out, int c_in,
                      std::vector<uint16_t> &wd, std::vector<uint32_t> &nz);
// dst[n][c][r] = src[n][r][c], floats, by tiles of 64 x 64.  A launch has fewer than 2^32 threads, 256 to a tile.
constexpr int64_t kTransposeMaxTiles = (1 << 24) - 1;
inline int64_t transpose_tiles(int64_t n, int64_t rows, int64_t cols) { return n * ((rows + 63) / 64) * ((cols + 63) / 64); }
int launch_transpose(const float *src, float *dst, int n, int rows, int cols, void *stream);
int launch_maxpool2x2(const void *x, void *y, int n, int c, int h, int w, int layout, int dtype,
                      void *stream);

}  // namespace pconv
