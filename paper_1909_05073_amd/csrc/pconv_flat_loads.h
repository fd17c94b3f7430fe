// Where pconv_mfma_flat.hip reads its pixels.  Plain C++, so that a host program can walk through all of it.
#pragma once

#include <cstdint>

namespace pconv {

// A buffer load at byte `lane` (per lane) + `uniform` (of the wave) of the input tensor.  Whether the hardware counts
// the uniform part when it checks an offset against the buffer's size is not relied on: a load that must not
// read has bit 31 of `lane` set (tensors are smaller than that) and a uniform part that lies in the tensor, and every
// other one lies in the tensor as a whole (in the dwords that hold it, where planes have odd numbers of pixels).
constexpr uint32_t kNoLoad = 0x80000000u;
struct FlatLoad { uint32_t lane, uniform; };
constexpr uint32_t lesser(uint32_t a, uint32_t b) { return a < b ? a : b; }

// Sixteen bytes of channel (channels last: pixel) j of an item: src is the item's first element in the step's first
// channel, c0 that channel, g_item the item's plane of eight channels.
template <bool NCHW, bool ODD>
constexpr FlatLoad flat_load(uint32_t src, int g_item, int j, int c0, int c_in, uint32_t plane_step)
{
    // (the sign of `left`: the channel is beyond the last one; channels last: c_in is a multiple of 8)
    const int left = c_in - 1 - (c0 + g_item * 8) - (NCHW ? j : 0);
    const uint32_t beyond = uint32_t(left) & kNoLoad;
    // (the uniform part of a channel beyond is that of the last one)
    if (!NCHW) return FlatLoad{src | beyond, uint32_t(lesser(uint32_t(c0), uint32_t(c_in - 1)) + uint32_t(j * c_in)) * 2u};
    // ODD: from the dword of the first element on (uniform + 2 * (j & 1) is a multiple of four: the blocks of
    // channels begin at even ones)
    const uint32_t odd = ODD ? 2u * uint32_t(j & 1) : 0u;
    return FlatLoad{(ODD ? (src + odd) & ~3u : src) | beyond,
                    lesser(uint32_t(c0) * plane_step + (uint32_t(j) * plane_step - odd), uint32_t(c_in - 1) * plane_step)};
}

// ODD: the dword behind those sixteen bytes.  Only an item that begins in the middle of a dword needs it; behind
// the last item of a tensor whose size is a multiple of four it would lie outside.
constexpr FlatLoad flat_load_fifth(FlatLoad row, uint32_t src, int j)
{
    return FlatLoad{row.lane | (~(src + 2u * uint32_t(j & 1)) & 2u) << 30, row.uniform + 16u};
}

}  // namespace pconv
