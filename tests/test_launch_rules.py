"""CPU tests of the rules that choose a launch by sizes alone (csrc/launch_rules.h), against points measured on both sides."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(expression) -> its integer value, in C++ with the rules at hand."""
    def run(*expressions):
        tmp = tmp_path_factory.mktemp("rules")
        src, exe = tmp / "ask.cpp", tmp / "ask"
        lines = "\n".join('    printf("%%d\\n", (int)(%s));' % e for e in expressions)
        src.write_text('#include "launch_rules.h"\n#include <cstdio>\nint main()\n{\n%s\n    return 0;\n}\n' % lines)
        subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2211_00839_amd", "csrc"), str(src), "-o", str(exe)],
                       check=True, timeout=60)
        out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True, timeout=60).stdout
        return [int(x) for x in out.split()]
    return run


def test_single_classes_are_cut_into_slices_only_where_that_is_faster(ask):
    # (samples, blocks, ms with one workgroup, ms in slices)
    measured = [(2561, 5, 9.7, 13.9), (2561, 8, 10.5, 14.7), (2900, 6, 11.0, 16.1), (3072, 5, 11.5, 16.8), (3072, 8, 12.5, 17.5),
                (3073, 5, 18.1, 16.9), (3073, 8, 20.0, 17.8), (3600, 5, 21.3, 20.7), (5120, 8, 35.2, 29.8), (2561, 9, 17.3, 15.7),
                (2561, 12, 18.2, 17.2), (2700, 16, 20.0, 19.2), (5120, 16, 41.6, 34.4), (5121, 1, 35.2, 32.3), (5121, 4, 39.4, 27.5),
                (5000, 4, 20.0, 28.0), (8000, 8, 75.9, 47.3)]
    first = ask(*["rules::sliced_from(1, %d)" % K for _, K, _, _ in measured])
    for (n, K, whole, sliced), least in zip(measured, first):
        assert (n >= least) == (sliced < whole), (n, K)


def test_recompute_sweeps_are_cut_into_pieces_only_where_that_is_faster(ask):
    # (classes, samples each, d, blocks, ms in pieces of 64 candidates, ms in wide tiles)
    measured = [
        # wide tiles to fill the device up to twice: long rows, few blocks and full tiles are better left wide
        (125, 500, 2048, 1, 606, 452), (125, 500, 2048, 2, 433, 340), (125, 500, 2048, 4, 214, 177), (125, 500, 2048, 16, 59.1, 51.6),
        (100, 500, 2048, 1, 526, 446), (100, 500, 2048, 4, 188, 174), (100, 500, 2048, 16, 51.9, 50.4), (90, 500, 2048, 2, 347, 332),
        (500, 250, 2048, 1, 380, 330), (55, 700, 2048, 1, 718, 665), (20, 1280, 2048, 1, 1267, 1087), (16, 1280, 2048, 2, 746, 700),
        (6, 2300, 2048, 1, 2047, 1898), (2, 3900, 2048, 1, 3248, 3052), (20, 1280, 2048, 4, 442, 416), (125, 500, 1024, 1, 266, 229),
        (110, 500, 1024, 2, 183, 170), (125, 500, 1024, 4, 95.7, 91.0), (100, 500, 1024, 1, 235, 225), (20, 1280, 1024, 1, 612, 572),
        (125, 500, 512, 1, 136, 124), (110, 500, 512, 2, 95.6, 92.9), (20, 1280, 512, 1, 324, 314),
        # the same range, other calls
        (100, 500, 512, 16, 15.2, 17.0), (100, 500, 512, 4, 46.8, 50.3), (50, 700, 512, 4, 63.9, 74.5), (300, 250, 1024, 1, 122, 158),
        (400, 250, 512, 4, 30.5, 38.9), (44, 700, 1024, 4, 110, 132), (75, 500, 2048, 4, 150, 171), (4, 2300, 512, 2, 300, 337),
        (36, 700, 1024, 1, 232, 253), (12, 1280, 512, 4, 86.7, 102.3), (2, 3000, 2048, 1, 1701, 1882), (100, 500, 32, 1, 25.7, 27.0),
        (75, 500, 4096, 1, 884, 869), (75, 500, 4096, 8, 167, 185), (56, 600, 768, 3, 97.8, 114.8), (125, 500, 256, 1, 76.4, 73.2),
        # at most one wide tile to a compute unit, and more than two
        (64, 500, 2048, 1, 304, 285), (64, 500, 4096, 1, 678, 570), (250, 250, 2048, 1, 182, 167), (16, 1000, 4096, 1, 1174, 1093),
        (64, 500, 4096, 3, 323, 330), (64, 500, 8192, 2, 1091, 902), (64, 500, 2048, 8, 60.0, 69.8), (1, 4000, 4096, 1, 3970, 4304),
        (1, 200, 32, 1, 5.39, 7.34), (1, 4096, 2048, 1, 2112, 2276), (10, 1000, 512, 4, 50.6, 72.5), (100, 250, 2048, 1, 89, 140),
        (6, 2500, 512, 4, 408, 406)]
    said = ask(*["rules::recompute_in_pieces([](int) { return %d; }, %d, %d, %d, 256)" % (n, L, d, K)
                 for L, n, d, K, _, _ in measured])
    for (L, n, d, K, pieces, wide), yes in zip(measured, said):
        assert bool(yes) == (pieces < wide), (L, n, d, K)
    # unequal classes are counted one by one: 243 wide tiles, 543
    assert ask("rules::recompute_in_pieces([](int i) { return i ? 1 : 3000; }, 100, 512, 4, 256)") == [1]
    assert ask("rules::recompute_in_pieces([](int i) { return i ? 1 : 3000; }, 400, 512, 4, 256)") == [0]
