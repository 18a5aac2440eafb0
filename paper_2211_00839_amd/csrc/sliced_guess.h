// How far the sliced step loop (sliced_kernels.hip) picks ahead.  A pick for a block that has one in the trip already is a guess;
// where samples come with near copies many fail, and a guess that fails costs its row and its lists (2 us) and drops the picks
// behind it.  Plain functions of words, so that they can be tested without a device.
#pragma once

namespace sliced {

// What a class knows of its guesses: the share that held lately in parts of GUESS_ONE, and in the low bits the trips since one was
// made.
constexpr int GUESS_ONE = 4096, GUESS_BITS = 4, GUESS_TRIPS = 4;
constexpr int GUESS_FIRST = GUESS_ONE << GUESS_BITS;
constexpr int GUESS_MOST = 7;      // of a trip: its picks but the first
// It lasts from launch to launch of a call (several classes: some twenty trips each), in memory that is zero when a call starts.
constexpr int guess_stored(int word) { return GUESS_FIRST - word; }
constexpr int guess_loaded(int stored) { return GUESS_FIRST - stored; }

// The most guesses of the next trip: as many as hold together in two trips of five (a step in a trip of its own takes about
// two and a half times what a pick takes); where one does not, one every GUESS_TRIPS trips to see whether that is still so.
constexpr int guesses_ahead(int word)
{
    const int share = word >> GUESS_BITS, trips = word & ((1 << GUESS_BITS) - 1);
    constexpr int at_least[GUESS_MOST] = {1638, 2591, 3018, 3257, 3410, 3516, 3593};      // GUESS_ONE times 0.4 to the power of 1 / m
    int most = 0;
    for (int m = 0; m < GUESS_MOST; ++m) most += share >= at_least[m] ? 1 : 0;
    return most == 0 && trips >= GUESS_TRIPS - 1 ? 1 : most;
}

// The word behind a trip with `held` guesses that held, and one at which it was cut or none.
constexpr int guess_after(int word, int held, bool cut)
{
    int share = word >> GUESS_BITS, trips = word & ((1 << GUESS_BITS) - 1);
    if (held == 0 && !cut) return trips < GUESS_TRIPS - 1 ? word + 1 : word;
    share += held * ((GUESS_ONE - share) >> 4);
    if (cut) share -= share >> 4;
    return share << GUESS_BITS;
}

// How many blocks the next trip looks at: twice as many as had picks that hold.
constexpr int blocks_after(int used, int most) { return 2 * used < most ? 2 * used : most; }

} // namespace sliced
