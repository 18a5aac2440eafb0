// Rules of a dispatch that are a matter of sizes alone: plain host code, so that the measured points behind them can be
// tested without a device.
#pragma once
#include <algorithm>
#include <cstdint>

namespace rules {

// Least samples in the largest class of a launch for the step loop that cuts classes into slices (sliced_kernels.hip).  Classes
// of more than four blocks are cut as soon as one workgroup's registers do not hold them: above 2560 samples with
// more than eight blocks, above 3072 with more than four (5120 fit, but too few registers are left).  One class of a mixture, one
// workgroup / slices, in ms: eight blocks 3072 samples 13.6 / 13.8, 3073 19.7 / 13.5, five blocks 3072 11.6 / 13.2, 3073 17.7 / 13.3, four
// 4000 16.0 / 16.7, 5000 20.7 / 20.1, 5121 39.4 / 20.5, one 4000 15.4 / 15.6, 5121 36.1 / 19.6; nine blocks 2561 16.6 / 12.8, sixteen 18.2 /
// 13.6 (and 2560 18.3 / 14.1: the line could lie lower there).  Several, one workgroup to a class and its
// helpers / slices: ten of 5000, four blocks 25.2 / 30.1, five 35.1 / 29.2, eight 39.8 / 31.0, sixteen 54.3 / 38.1, ten of 4000, eight 29.8 /
// 23.4, ten of 2600, sixteen 23.1 / 19.3, 60 of 3500, eight 39.0 / 37.8, 60 of 4000, five 39.4 / 38.2; thirty of 3000, eight 18.0 /
// 24.0, ten of 2000, sixteen 10.4 / 13.8.
// wide: in slices of more than 1024 samples.  Several classes, of 2048: 80 of 3500, eight blocks 47.1 / 52.5, 100 of 5000, eight
// 107 / 121, 100 of 3000, sixteen 58.9 / 63.3 (100 of 4000, eight 69.8 / 66.9).
constexpr int SLICED_ALWAYS_FROM = 5121;
constexpr int sliced_from(int classes, int K, bool wide = false)
{
    if (wide && classes > 1) return SLICED_ALWAYS_FROM;
    return K > 8 ? 2561 : K > 4 ? 3073 : SLICED_ALWAYS_FROM;
}

// Whether the classes that are cut, those of `least` samples and more, are enough of the work of a launch of several smaller ones: a
// quarter of it or more.  One workgroup to a class / slices, eight blocks, in ms: one of 5000 beside forty of 500 33.9 / 25.5; of 3500
// beside forty of 2000 27.0 / 27.7.  size(i) = samples of class i of `classes`.
template <typename Size> bool enough_is_cut(const Size &size, int classes, int least)
{
    int largest = 0;
    double cut = 0.0, work = 0.0;
    for (int i = 0; i < classes; ++i) {
        const int n = size(i);
        const double mine = (double)n * n;
        largest = std::max(largest, n);
        work += mine;
        if (n >= least) cut += mine;
    }
    return classes == 1 || largest >= SLICED_ALWAYS_FROM || 4.0 * cut >= work;
}

// The slices of the classes of a launch: at least `least` samples each, at most `most` of them to a class.
// slice(i) gets the samples of class i's slices, a multiple of 256; none is empty.  Their number in all, and the largest and the most.
struct Slices {
    int count, largest, most;
};
template <typename Pitch, typename Slice> Slices slices(const Pitch &pitch, int classes, int least, int most, const Slice &slice)
{
    Slices out = {0, 0, 0};
    for (int i = 0; i < classes; ++i) {
        const int ld = pitch(i);
        int W = std::min(most, (ld + least - 1) / least);
        const int seg = ((ld + W - 1) / W + 255) / 256 * 256;
        W = (ld + seg - 1) / seg;
        slice(i, seg, W);
        out.count += W;
        out.largest = std::max(out.largest, seg);
        out.most = std::max(out.most, W);
    }
    return out;
}

// What the sliced loops hold: samples of a slice, slices of a class, the same in slices of more than 1024 samples with more than
// eight blocks (another loop, whose exchange area holds fewer).
constexpr int SLICE_WIDEST = 2048, SLICES_MOST = 64, SLICES_MOST_PAIRS = 32;

// 0 where the classes of a launch are not cut into slices, else the least samples of a slice: 1024 where there are compute units for
// that, one workgroup to a unit, else 2048.  min_n, wide_n: sliced_from() without and with `wide` (no matter for one class); given: samples of a slice, 0 to
// choose; most, most_pairs: slices of a class at most; wgs: workgroups of the launch at most.
template <typename Size, typename Pitch>
int slice_least(const Size &size, const Pitch &pitch, int classes, int K, int cus, int min_n, int wide_n, int given = 0,
                int most = SLICES_MOST, int most_pairs = SLICES_MOST_PAIRS, int wgs = 1 << 30)
{
    int max_n = 0;
    for (int i = 0; i < classes; ++i) max_n = std::max(max_n, (int)size(i));
    if (min_n == 0 || max_n < min_n || cus / classes < 2 || max_n > 1024 * SLICES_MOST) return 0;
    if (!enough_is_cut(size, classes, min_n)) return 0;
    for (const int least : {given ? given : 1024, given ? given : SLICE_WIDEST}) {
        const int per_class = std::min(least > 1024 && K > 8 ? most_pairs : most, cus / classes);
        if (per_class < 2) return 0;
        const Slices cut = slices(pitch, classes, least, per_class, [](int, int, int) {});
        if (cut.largest > 1024 && !given && max_n < wide_n) return 0;
        if (cut.count > std::min(cus, wgs) || cut.largest > SLICE_WIDEST) continue;
        if (cut.largest > 1024 && K > 8 && cut.most > SLICES_MOST_PAIRS) continue;
        return least;
    }
    return 0;
}

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
