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
