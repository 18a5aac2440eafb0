"""CPU test of how far the sliced step loop picks ahead (csrc/sliced_guess.h): where guesses fail, few are made, where they hold,
all of them, and a class whose guesses come to hold is noticed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "sliced_guess.h"
#include <cstdio>
#include <random>

using namespace sliced;
#define EXPECT(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

static std::mt19937 rng(3);
static int word = GUESS_FIRST;

struct Run { long made, held; };
// trips of one block: every guess of a trip holds with that chance, the first that does not ends the trip
static Run trips(int count, double chance)
{
    Run r = {0, 0};
    for (int t = 0; t < count; ++t) {
        const int made = guesses_ahead(word);
        int held = 0;
        while (held < made && std::uniform_real_distribution<double>(0, 1)(rng) < chance) ++held;
        word = guess_after(word, held, held < made);
        r.made += made;
        r.held += held;
    }
    return r;
}

int main()
{
    EXPECT(guesses_ahead(GUESS_FIRST) == 7);
    EXPECT(guess_loaded(0) == GUESS_FIRST);              // a call starts with zeroed memory
    Run r = trips(1000, 1.0);
    EXPECT(r.made == 7000);
    r = trips(10000, 0.99);
    EXPECT(r.made > 6.7 * 10000);                        // one in a hundred fails: hardly fewer
    r = trips(10000, 0.5);
    EXPECT(r.made < 1.2 * 10000 && r.made > 0.4 * 10000);
    trips(40, 0.0);
    r = trips(8000, 0.0);
    EXPECT(r.made == 8000 / GUESS_TRIPS);                              // none hold: one in GUESS_TRIPS trips
    trips(80, 1.0);
    EXPECT(guesses_ahead(word) == 7);                    // and all again when they do
    // whatever comes, the word stays a share and a count of trips, and no trip has more than seven
    for (int it = 0; it < 100000; ++it) {
        word = guess_after(word, (int)(rng() % 8), rng() % 2 != 0);
        EXPECT((word >> GUESS_BITS) >= 0 && (word >> GUESS_BITS) <= GUESS_ONE);
        EXPECT((word & ((1 << GUESS_BITS) - 1)) < GUESS_TRIPS);
        EXPECT(guess_loaded(guess_stored(word)) == word);
        EXPECT(guesses_ahead(word) >= 0 && guesses_ahead(word) <= 7);
    }
    // blocks: one after a trip that served one, all of them again in three trips
    EXPECT(blocks_after(1, 8) == 2 && blocks_after(4, 8) == 8 && blocks_after(8, 8) == 8);
    return 0;
}
"""


def test_guesses_are_made_where_they_hold(tmp_path):
    src, exe = tmp_path / "guess.cpp", tmp_path / "guess"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2211_00839_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
