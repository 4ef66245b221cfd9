// Index division and launch rules of the row quantizers: plain C++ without HIP types, so that they can be compiled and exercised
// on their own (tests build them with the address and undefined-behaviour sanitizers).  Kernels call the constexpr functions.
#ifndef NVFP4_QUANTIZE_PLAN_H
#define NVFP4_QUANTIZE_PLAN_H

#include <algorithm>
#include <cstdint>

namespace nvfp4 {

// Division of indexes by a width that a whole launch shares (blocks of a row, heads): one 32 x 32-bit multiplication and a
// shift with a factor that the host computes, where a division by a run-time number is twenty to a hundred and more vector
// instructions.  The all-to-all order takes three of them a block, beside the 75 of the encoding, padded rows one (us, replayed
// from a graph, the same grids, divided -> multiplied: all-to-all order of 4620x24x128 in one launch 16.5 -> 15.2, in two passes
// 0.4 M blocks 11.0 -> 10.4, 0.7 M 14.2 -> 13.5, 3.5 M 48.5 -> 45.6; padded rows 3.5 M 45.5 -> 44.3, with the search 57.1 -> 55.8).
// Exact for n < 2^31: with l = ceil(log2 d) and m = ceil(2^(31+l) / d) < 2^32, m d exceeds
// 2^(31+l) by less than d, so n m / 2^(31+l) exceeds n / d by less than 1 / d (Granlund and Montgomery).
// m = 0: indexes may be larger, plain division.
constexpr uint32_t quotient(uint32_t n, uint32_t m, int shift) { return (uint32_t)(((uint64_t)n * m) >> shift); }
struct Divisor {
    uint32_t m = 0;
    int shift = 31;
    Divisor() = default;
    constexpr Divisor(int64_t divisor, int64_t indexes)         // every n divided is below `indexes`
    {
        if (divisor < 1 || divisor >= (1ll << 31) || indexes > (1ll << 31)) return;
        int l = 0;
        while ((1ll << l) < divisor) ++l;
        shift = 31 + l;
        m = (uint32_t)((((uint64_t)1 << shift) + (uint64_t)divisor - 1) / (uint64_t)divisor);
    }
    constexpr uint32_t small(uint32_t n) const { return quotient(n, m, shift); }
};
constexpr int64_t divide(int64_t n, int64_t divisor, const Divisor &by)
{
    return by.m ? (int64_t)by.small((uint32_t)n) : n / divisor;
}

// Workgroups of 256 lanes of a pass that encodes rows of `nblk` blocks of 16 elements.
// With partial maxima: four blocks to a lane, so that what every workgroup does first (the partial maxima again, the scale's tie
// tests: about as many vector instructions as a plain block) is paid once for four blocks, but at least kQuantMinGrid
// workgroups (four to a compute unit), or one block a lane where there are fewer.  With one block a lane up to the largest
// grid: 3520x24x128, smoothed keys and values with the search 31.0 us -> 30.0; 3520x3072 and 3520x14336
// in front of their GEMMs 0.6 us and 4 us less.  Two blocks a lane changed nothing (31.0), at least 768 workgroups less
// (30.5), 2048 as much (30.0); at most 1024 or 2048 for every size cost the 505 MB gradient 8 us.
// The plain rule keeps two blocks in flight a lane (the search one), and from kQuantLarge blocks on, where two blocks a lane
// are at least 2930 workgroups, two are as good or better: one turn a lane, nothing waits for a second fetch.  Whole call
// in two passes, us, one / two / four blocks a lane: 0.7 M 12.6 / 12.4 / 11.9, 0.9 M 15.2 / 14.7 / 14.2, 1.2 M 17.6 / 17.2 / 16.8,
// 1.7 M 23.3 / 22.9 / 23.4, 3.5 M 43.1 / 42.0 / 42.6, 5.0 M 58.7 / 58.1 / 58.9, 8.1 M 93.6 / 92.3 / 94.3, 10 M 122.1 / 122.3 / 123.4,
// 15.8 M 193.6 / 193.6 / 192.7; rows of a wider buffer the same within 0.3 us but for 1.7 M, 24.2 / 23.4 / 23.0.  With the
// search four throughout: 1.7 M 28.2 / 26.9 / 26.6, 3.5 M 52.2 / 49.0 / 47.8, 8.1 M 106 / 106 / 102, from 12 M on even.
// With a given scale there are no maxima to reduce, and one block a lane, up to the largest grid, has the most loads in
// flight (us, one / four blocks a lane; replayed from a graph on inputs in turn that exceed the 256 MB
// Infinity Cache): plain 0.7 M 7.0 / 7.0, 1.2 M 10.0 / 11.0, 1.7 M 13.6 / 14.8, 3.5 M 25.9 / 27.5, 5.0 M 36.3 / 39.0, 8.1 M
// 58.7 / 60.5, 12 M 87.5 / 88.8; with the search 1.2 M 11.6 / 12.9, 3.5 M 28.7 / 29.1, 5.0 M 41.0 / 40.7, 8.1 M 63 / 63.
constexpr int kQuantMaxGrid = 16384, kQuantMinGrid = 1024, kQuantBlocksPerLane = 4, kQuantLarge = 1500000;

inline int encode_rows_grid(int64_t nblk, bool given_scale, bool search)
{
    const int64_t per_lane = given_scale ? 1 : !search && nblk >= kQuantLarge ? 2 : kQuantBlocksPerLane;
    const int64_t all = (nblk + 255) / 256, few = (nblk + 256 * per_lane - 1) / (256 * per_lane);
    return (int)std::min<int64_t>(kQuantMaxGrid, std::max<int64_t>(few, std::min<int64_t>(all, kQuantMinGrid)));
}

// Whether a tensor that fits on the chip takes the one-launch form (the figures stand in nvfp4_quantize_resident.hip).
// library_scratch: the two passes would keep their partial maxima in the library's one array per GPU, where calls that overlap
// race, while the exchange words of the one-launch form are one of 64 sets; such calls keep the lower bound, at which
// the two forms are within a microsecond (on the device 0.80 M 14.2 us and 13.3, 0.89 M 14.7 and 13.9).
constexpr int64_t kOneLaunchBelow = 12000, kOneLaunchFrom = 950000, kOneLaunchFromScratch = 800000;

inline bool one_launch_pays(int64_t nblk, bool search, bool smooth, bool library_scratch)
{
    return !search && !smooth && (nblk < kOneLaunchBelow || nblk >= (library_scratch ? kOneLaunchFromScratch : kOneLaunchFrom));
}

}  // namespace nvfp4
#endif
