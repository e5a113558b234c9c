// Row lines of the unstructured selection: what unstructured_rows.hip (rows read twice) and unstructured_held.hip (rows
// held in registers) share.
#pragma once

#include "select.h"
#include "unstructured_tiled.h"

namespace dass {
namespace rowl {

constexpr int kRows = kRowlinesBlock;   // rows per workgroup
constexpr int kThreads = 1024;
constexpr int kBins = 256;
// Counters of a row: [0 .. 255] the bins ascending, then 64 counters for scores above the window and 64
// for scores below it, one per lane: a fifth of a row's scores lies on either side, and 64 lanes
// adding to one LDS word take turns.
constexpr int kAbove = kBins, kBelow = kBins + 64;
constexpr int kStride = kBins + 128;
constexpr int kSamples = 128;
constexpr int kCap = 256;               // listed scores per row
constexpr uint32_t kInfBits = 0x7f800000u;

struct Window {
    uint32_t lo, sh;
};
struct Select {
    uint32_t lo, width, need, inside;
};

__device__ __forceinline__ uint32_t mono(float q)   // unsigned integer that grows with q
{
    const uint32_t b = __float_as_uint(q);
    return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}

// The 128 sampled positions of a row are 16 runs of 8 consecutive columns (a sample spread one by one
// would touch 128 of the row's 172 memory lines: most of the matrix, just to sample it): run k
// lies in the k-th sixteenth of the row, at an offset that changes from run to run.  Returns the
// run's first column, a multiple of 8.
constexpr int kRuns = kSamples / 8;
__device__ __forceinline__ uint32_t sample_run(uint32_t k, uint32_t cols)
{
    const uint32_t octets = cols / 8, stratum = octets / kRuns;   // cols >= 1024: stratum >= 8
    const uint32_t o = (uint32_t)(((uint64_t)k * octets) / kRuns) + ((k * 2654435761u) >> 8) % stratum;
    return (o < octets ? o : octets - 1) * 8;
}

}  // namespace rowl
}  // namespace dass
