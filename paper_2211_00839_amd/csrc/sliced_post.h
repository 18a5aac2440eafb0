// What a workgroup's second post of a trip says in the sliced step loop (sliced_kernels.hip): the lengths of its segments of up to
// eight lists and, where they are few, the entries themselves.  Plain functions of words, so that they can be tested without a device.
#pragma once

namespace sliced {

constexpr int BM = 8;              // most picks of a trip
constexpr int POST = 16;           // 16-byte pieces of a workgroup's post
constexpr int ENTRIES = 1024;      // list entries that are applied in one trip, at most
// An entry on its way carries its pick and its place in the pick's segment above the sample's number.
constexpr int J_BITS = 17;
constexpr int SLICE_SAMPLES = 2048;     // of the largest slice: a length has twelve bits

// Piece 0: eight lengths of 12 bits in three words.
constexpr unsigned post_word0(int l0, int l1, int l2) { return (unsigned)l0 | (unsigned)l1 << 12 | (unsigned)l2 << 24; }
constexpr unsigned post_word1(int l2, int l3, int l4, int l5)
{
    return (unsigned)l2 >> 8 | (unsigned)l3 << 4 | (unsigned)l4 << 16 | (unsigned)l5 << 28;
}
constexpr unsigned post_word2(int l5, int l6, int l7) { return (unsigned)l5 >> 4 | (unsigned)l6 << 8 | (unsigned)l7 << 20; }
// Length u of them.
constexpr int post_length(int u, unsigned x, unsigned y, unsigned z)
{
    return u == 0   ? (int)(x & 0xFFF)
           : u == 1 ? (int)(x >> 12 & 0xFFF)
           : u == 2 ? (int)(x >> 24 | (y & 0xF) << 8)
           : u == 3 ? (int)(y >> 4 & 0xFFF)
           : u == 4 ? (int)(y >> 16 & 0xFFF)
           : u == 5 ? (int)(y >> 28 | (z & 0xFF) << 4)
           : u == 6 ? (int)(z >> 8 & 0xFFF)
                    : (int)(z >> 20);
}
// How many entries follow in a post whose lengths add up to `all`: all of them, or none where they do not fit and are in memory.
constexpr int entries_in_post(int all) { return all < POST ? all : 0; }
// What may be made of a length or a count that a post names: nothing if not all posts have come (the bounded wait ran out).  The
// words may be those of an earlier trip or torn then, and no place in the lists may be taken from them.
constexpr int believed(bool come, int count) { return come ? count : 0; }

constexpr int entry_word(int j, int pick, int place) { return j | pick << J_BITS | place << (J_BITS + 3); }
constexpr int entry_pick(int word) { return (word >> J_BITS) & (BM - 1); }
constexpr int entry_place(int word) { return (int)((unsigned)word >> (J_BITS + 3)); }
constexpr int entry_sample(int word) { return word & ((1 << J_BITS) - 1); }

} // namespace sliced
