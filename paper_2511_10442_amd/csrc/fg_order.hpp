// Lists and areas of the ordering of dense cells (fg_order.hip), filled by the prefix sum of the binning.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fg {

// Cells of more points than this are ordered.  Points of strongly varying density, binning + query + backward for 48 / 96 / 192, in us: 1.1M in one split,
// K = 16 1244 / 1237 / 1220; 2M in four, K = 8 1535 / 1471 / 1476, K = 16 1685 / 1625 / 1616; 5M in five, K = 8 3658 / 3560 / 3506, K = 16 3986 / 3922 / 3901.
constexpr int kOrderMin = 96;
constexpr int kOrderWindowShift = 10;
constexpr int kOrderChunk = 2 << kOrderWindowShift;      // points sorted in LDS at a time

// words of `counters`
constexpr int kOrderSmall = 0, kOrderLarge = 1, kOrderChunks = 2;

// Everything but bounds and coords lies in areas that the binning and the query stage use at other times.
struct OrderArgs {
    const float* coords;       // [n][d]
    const int32_t* bounds;     // cell boundaries
    float4* rec;               // [n] records
    int32_t* rows0;            // [n] rows of the pieces of even levels
    int32_t* rows1;            // [n] of the odd ones
    int32_t* counters;         // [3] zero before the prefix sum
    int32_t* small;            // cells of kOrderMin + 1 .. kOrderChunk points: less than n / 64
    int32_t* large;            // of more: less than n / 2048
    int32_t* stack;            // n / 256 + 1 words
    int4* chunks;              // of split pieces: first position, points, which rows.  A piece of L points has at most L / 1024 + 1 runs of small
                               // sub-cells, and m / 2048 + 1 parts of a larger one of m > 1024: 3.5 n / 1024 for each of eight levels
};

// The lists inside an area of n words (n >= 2^15): at most n / 64, n / 2048, n / 256 + 1 and 4 * 28 n / 1024 of them.
inline OrderArgs order_args(const float* coords, const int32_t* bounds, float* rec, int32_t* rows0, int32_t* rows1, int32_t* counters, int32_t* area,
                            int64_t n)
{
    OrderArgs a;
    a.coords = coords; a.bounds = bounds; a.rec = reinterpret_cast<float4*>(rec);
    a.rows0 = rows0; a.rows1 = rows1; a.counters = counters;
    a.small = area;
    a.large = area + n / 16;
    a.stack = area + n / 8;
    a.chunks = reinterpret_cast<int4*>(area + n / 4 / 4 * 4);
    return a;
}

// two dimensions only: elsewhere nothing that searches by boxes has gained from it
hipError_t launch_order(const OrderArgs& a, hipStream_t stream);

}  // namespace fg
