// Walks through every pixel load that the flat matrix-core kernel can issue for a set of small tensors and reports
// those that leave the tensor, or that a size check on the per-lane offset alone would let through, or that miss
// an element.  See test_flat_loads.py.
#include <cstdio>
#include <initializer_list>

#include "pconv_flat_loads.h"

using namespace pconv;

static long bad = 0, seen = 0;

template <bool NCHW, bool ODD>
static void walk(int n, int c_in, int hw, uint32_t lead, int kb)
{
    const uint32_t x_bytes = uint32_t(n) * c_in * hw * 2, plane_step = uint32_t(hw) * 2;
    const uint32_t size = ODD ? (lead + x_bytes + 3) & ~3u : x_bytes;          // of the buffer, from x - lead on
    const int step = 16 * kb;
    auto check = [&](FlatLoad at, uint32_t bytes, const char *what, int j, int c0, int g) {
        ++seen;
        const bool refused = at.lane >= kNoLoad;
        const bool inside = !refused && uint64_t(at.lane) + at.uniform + bytes <= size;
        if ((refused && at.uniform > x_bytes) || (!refused && !inside)) {
            if (++bad < 5)
                std::printf("%s: n=%d c_in=%d hw=%d lead=%u kb=%d j=%d c0=%d plane=%d: offset %u + %u, %u bytes, buffer %u\n", what, n,
                            c_in, hw, lead, kb, j, c0, g, at.lane, at.uniform, bytes, size);
        }
    };
    for (int img = 0; img < n; ++img)
        for (int q = 0; q < hw; q += 8) {
            const int q8 = q + 8 <= hw ? q : hw - 8;
            for (int c0 = 0; c0 < c_in + 20 * step; c0 += step)
                for (int g = 0; g < 2 * kb; ++g)
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t e = NCHW ? uint32_t(img * c_in * hw + q8) : uint32_t((img * hw + q8) * c_in);
                        const uint32_t src = e * 2 + (NCHW ? plane_step : 2u) * 8u * uint32_t(g) + lead;
                        const FlatLoad at = flat_load<NCHW, ODD>(src, g, j, c0, c_in, plane_step);
                        check(at, 16, "row", j, c0, g);
                        const int c = c0 + g * 8 + (NCHW ? j : 0);
                        if ((c < c_in) == (at.lane >= kNoLoad)) { ++bad; std::printf("channel %d of %d\n", c, c_in); }
                        const FlatLoad behind = flat_load_fifth(at, src, j);
                        if (ODD) check(behind, 4, "behind", j, c0, g);
                        if (c >= c_in) continue;
                        // the item's sixteen bytes are among those read
                        const uint64_t first = lead + 2 * (NCHW ? (uint64_t(img) * c_in + c) * hw + q8 : (uint64_t(img) * hw + q8 + j) * c_in + c);
                        const uint64_t from = uint64_t(at.lane) + at.uniform;
                        const uint64_t to = from + (ODD && behind.lane < kNoLoad ? 20 : 16);
                        if (first < from || first + 16 > to) { ++bad; std::printf("item at %llu, read %llu to %llu\n", (unsigned long long)first, (unsigned long long)from, (unsigned long long)to); }
                    }
        }
}

int main()
{
    for (int kb : {1, 2})
        for (int n : {1, 3})
            for (int c_in : {1, 2, 7, 8, 16, 24, 33, 64, 512}) {
                for (int hw : {9, 15, 49, 63})
                    for (uint32_t lead : {0u, 2u}) walk<true, true>(n, c_in, hw, lead, kb);
                for (int hw : {8, 10, 56, 64}) walk<true, false>(n, c_in, hw, 0, kb);
                if (c_in % 8 == 0)
                    for (int hw : {8, 9, 49}) walk<false, false>(n, c_in, hw, 0, kb);
            }
    std::printf("%ld of %ld loads are wrong\n", bad, seen);
    return bad != 0 || seen == 0;
}
