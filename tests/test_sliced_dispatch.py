"""CPU test of which launches are cut into slices (csrc/launch_rules.h: slice_least()), against points measured on both sides: calls on
mixtures of 64 features, one workgroup to a class and its helpers / slices, on 256 compute units."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# (sizes as (count, samples), blocks, ms with one workgroup, ms in slices)
MEASURED = [
    ([(10, 5000)], 4, 25.2, 30.1), ([(10, 5000)], 5, 35.1, 29.2), ([(10, 5000)], 8, 39.8, 31.0), ([(10, 5000)], 16, 54.3, 38.1),
    ([(10, 4000)], 8, 29.8, 23.4), ([(10, 2600)], 16, 23.1, 19.3), ([(60, 3500)], 8, 39.0, 37.8), ([(60, 4000)], 5, 39.4, 38.2),
    ([(30, 3000)], 8, 18.0, 24.0), ([(10, 2000)], 16, 10.4, 13.8),
    # classes that are cut beside smaller ones: a quarter of the work or less
    ([(1, 5000), (40, 500)], 8, 33.9, 25.5), ([(1, 3500), (40, 2000)], 8, 27.0, 27.7),
    # only in slices of 2048
    ([(80, 3500)], 8, 47.1, 52.5), ([(100, 5000)], 8, 107.0, 121.0), ([(100, 3000)], 16, 58.9, 63.3),
    # one class
    ([(1, 3072)], 8, 13.6, 13.8), ([(1, 3073)], 8, 19.7, 13.5), ([(1, 3072)], 5, 11.6, 13.2), ([(1, 3073)], 5, 17.7, 13.3),
    ([(1, 4000)], 4, 16.0, 16.7), ([(1, 5121)], 4, 39.4, 20.5), ([(1, 4000)], 1, 15.4, 15.6), ([(1, 5121)], 1, 36.1, 19.6),
    ([(1, 2561)], 9, 16.6, 12.8), ([(1, 2561)], 12, 17.4, 13.1), ([(1, 2561)], 16, 18.2, 13.6),
]

# (sizes, blocks, samples of the largest slice; 0: not cut)
EDGES = [([(1, 50000)], 8, 1024), ([(1, 65536)], 16, 1024), ([(1, 65537)], 8, 0), ([(40, 12000)], 8, 2048), ([(16, 20000)], 16, 1280),
         ([(128, 6000)], 4, 0), ([(129, 6000)], 4, 0), ([(42, 6000)], 4, 1024), ([(43, 6000)], 4, 1280), ([(1, 6000), (30, 500)], 4, 1024),
         ([(1, 4000), (200, 300)], 8, 0)]

PROGRAM = r"""
#include "launch_rules.h"
#include <cstdio>
#include <utility>
#include <vector>

static int ask(std::vector<std::pair<int, int>> parts, int K)
{
    std::vector<int> n;
    for (auto p : parts) n.insert(n.end(), p.first, p.second);
    const int classes = (int)n.size();
    auto pitch = [&](int i) { return (n[i] + 255) / 256 * 256; };
    const int least = rules::slice_least([&](int i) { return n[i]; }, pitch, classes, K, 256, rules::sliced_from(classes, K),
                                         rules::sliced_from(classes, K, true));
    if (least == 0) return 0;
    // slices cover their class, none is empty, and no more of them than one to a compute unit
    const int most = least > 1024 && K > 8 ? rules::SLICES_MOST_PAIRS : rules::SLICES_MOST;
    bool good = true;
    const rules::Slices cut = rules::slices(pitch, classes, least, most < 256 / classes ? most : 256 / classes, [&](int i, int seg, int W) {
        good = good && seg %% 256 == 0 && seg * W >= pitch(i) && seg * (W - 1) < pitch(i) && W <= most && seg <= rules::SLICE_WIDEST;
    });
    return good && cut.count <= 256 ? cut.largest : -1;
}

int main()
{
%s
    return 0;
}
"""


def ask(tmp_path, launches):
    lines = ["    printf(\"%%d\\n\", ask({%s}, %d));" % (", ".join("{%d, %d}" % p for p in parts), K) for parts, K in launches]
    src, exe = tmp_path / "ask.cpp", tmp_path / "ask"
    src.write_text(PROGRAM % "\n".join(lines))
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2211_00839_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, timeout=120)
    out = subprocess.run([str(exe)], check=True, stdout=subprocess.PIPE, text=True, timeout=60).stdout
    return [int(x) for x in out.split()]


def test_launches_are_cut_into_slices_only_where_that_is_faster(tmp_path):
    said = ask(tmp_path, [(parts, K) for parts, K, _, _ in MEASURED])
    for (parts, K, whole, sliced), largest in zip(MEASURED, said):
        assert largest >= 0 and (largest > 0) == (sliced < whole), (parts, K, largest)


def test_the_edges_of_what_the_sliced_loops_hold(tmp_path):
    said = ask(tmp_path, [(parts, K) for parts, K, _ in EDGES])
    assert said == [largest for _, _, largest in EDGES]
