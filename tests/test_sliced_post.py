"""CPU test of the posts in which the workgroups of a sliced class tell one another their lists (csrc/sliced_post.h): what is packed
comes out again up to the largest slice, and a post that has not come (the bounded wait ran out: its words may be anything) names no
entry that could be given a place."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "sliced_post.h"
#include <cstdio>
#include <random>

using namespace sliced;
#define EXPECT(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main()
{
    std::mt19937 rng(5);
    auto upto = [&](int most) { return (int)(rng() % (unsigned)(most + 1)); };
    for (int it = 0; it < 20000; ++it) {
        const int most = it % 3 == 0 ? 2 : it % 3 == 1 ? SLICE_SAMPLES : 40;
        int len[BM], all = 0;
        for (int u = 0; u < BM; ++u) all += len[u] = it == 1 ? SLICE_SAMPLES : it % 7 == 0 && u > 1 ? 0 : upto(most);
        const unsigned x = post_word0(len[0], len[1], len[2]), y = post_word1(len[2], len[3], len[4], len[5]);
        const unsigned z = post_word2(len[5], len[6], len[7]);
        for (int u = 0; u < BM; ++u) EXPECT(believed(true, post_length(u, x, y, z)) == len[u]);
        EXPECT(entries_in_post(all) == (all < POST ? all : 0));
        // any words at all: no length and no entry is believed of posts that have not come
        int any = 0;
        for (int u = 0; u < BM; ++u) {
            const int l = post_length(u, rng(), rng(), rng());
            EXPECT(l >= 0 && l < 4096 && believed(false, l) == 0);
            any += l;
        }
        EXPECT(believed(false, entries_in_post(any)) == 0);
        // an entry of a post has one of the first POST - 1 places of its segment
        const int j = upto((1 << J_BITS) - 1), u = upto(BM - 1), place = upto(POST - 2), w = entry_word(j, u, place);
        EXPECT(entry_sample(w) == j && entry_pick(w) == u && entry_place(w) == place);
    }
    return 0;
}
"""


def test_posts_of_lists(tmp_path):
    src, exe = tmp_path / "post.cpp", tmp_path / "post"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover", "-I",
                    os.path.join(ROOT, "paper_2211_00839_amd", "csrc"), str(src), "-o", str(exe)], check=True, timeout=60)
    subprocess.run([str(exe)], check=True, timeout=60)
