// Rules of a dispatch that are a matter of sizes alone: plain host code, so that the measured points behind them can be
// tested without a device.
#pragma once
#include <algorithm>
#include <cstdint>

namespace rules {

// Least samples in the largest class of a launch for the step loop that cuts classes into slices (sliced_kernels.hip).  Classes
// of more than four blocks are cut as soon as one workgroup's registers do not hold them: above 2560 samples with
// more than eight blocks, above 3072 with more than four (5120 fit, but too few registers are left).  One class, one
// workgroup / slices with two picks to a trip, in ms: eight blocks 3072 samples 12.5 / 17.5, 3073 20.0 / 17.8, five blocks 3072
// 11.5 / 16.8, 3073 18.1 / 16.9, twelve blocks 2561 18.2 / 17.2, sixteen 19.0 / 17.2.  Several, one workgroup to a class and its
// helpers / slices with up to eight picks to a trip: ten of 5000, four blocks 25.5 / 31.9, five 34.6 / 31.0, eight 40.4 / 32.0, sixteen
// 54.4 / 38.1, ten of 4000, eight 31.1 / 23.9, ten of 2600, sixteen 23.4 / 19.3, 60 of 3500, eight 39.1 / 37.2, 60 of 4000, five
// 39.1 / 39.4; thirty of 3000, eight 18.0 / 24.0, ten of 2000, sixteen 10.6 / 14.5.
constexpr int sliced_from(int /*classes*/, int K) { return K > 8 ? 2561 : K > 4 ? 3073 : 5121; }

// Below that many samples several classes are cut only where the device holds them in slices of 1024: in slices of 2048, 80 of
// 3500, eight blocks 47.1 / 52.5, 100 of 5000, eight 107 / 121, 100 of 3000, sixteen 58.9 / 63.3 (100 of 4000, eight 69.8 / 66.9).
constexpr int SLICED_WIDE_FROM = 5121;

// Whether a recompute sweep (fp32) is better cut into pieces of 64 candidates than into tiles of 256 x 256: size(i) = samples of
// class i of `classes`, features of d values, K blocks, a device of `cus` compute units.
// A compute unit runs one wide tile or two pieces at a time, and a piece is a quarter of a tile's work.  Pieces lie closer
// round the candidates that are left, and their last round is less empty; but they read their operands from memory without
// sharing them through LDS, which costs more per product, and more again the less of the features the last-level cache (256 MB)
// holds.  So the rounds of both over the course of a call are counted (the classes have equal shares left; at least one
// round) and held against what a product costs more: the first number is for one block, two or three, and more (the fewer blocks, the
// more sweeps a step).  Pieces / wide measured, whole calls in ms: 100 classes of 500 and sixteen blocks, d = 512 15.2 / 17.0, d = 2048
// 51.9 / 50.4 and one block 526 / 446; 125 of 500, d = 2048, four 214 / 177; 20 of 1280, one block, d = 512 324 / 314, d = 128
// 114 / 118; ten of 1000, d = 512, four 51 / 73.  Up to one wide tile to a unit, pieces were faster wherever measured with more
// than one block (64 of 500, d = 4096, three 323 / 330; d = 8192, two 1091 / 902); with one, 64 of 500 and d = 2048 304 / 285, one class of 4096 2112 / 2276.
template <typename Size> bool recompute_in_pieces(const Size &size, int classes, int64_t d, int K, int cus)
{
    auto per = [](int64_t n, int64_t width) { return (n + width - 1) / width; };
    int64_t first = 0, samples = 0;
    for (int i = 0; i < classes; ++i) {
        first += per(size(i), 256) * per(size(i), 256);
        samples += size(i);
    }
    if (first > 2 * cus) return false;
    if (first <= cus && K > 1 && d <= 4096) return true;
    constexpr int POINTS = 16;               // of a call's course
    int64_t wide = 0;                        // rounds of wide tiles
    double pieces = 0.0;                     // the pieces' work in the same measure
    for (int p = 1; p <= POINTS; ++p) {
        int64_t w = 0, q = 0;
        for (int i = 0; i < classes; ++i) {
            const int64_t left = per((int64_t)size(i) * p, POINTS), rows = per(size(i), 256);
            w += per(left, 256) * rows;
            q += per(left, 64) * rows;
        }
        wide += per(w, cus);
        pieces += (double)std::max<int64_t>(q, 2 * cus) / (4 * cus);
    }
    const double megabytes = (double)samples * (double)d * 4.0 / (1 << 20);
    const double dearer = (K == 1 ? 1.41 : K <= 3 ? 1.37 : 1.25) + std::min(megabytes, K == 1 ? 500.0 : 300.0) / 700.0;
    return dearer * pieces <= (double)wide;
}

} // namespace rules
