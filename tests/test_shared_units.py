"""CPU test of the count of compute units (csrc/shared_units.h) that calls whose workgroups wait for one another take their
units from: the sum never exceeds the device, who does not fit waits until units are given back, and nobody is passed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "shared_units.h"
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

static void pause_ms(int ms) { std::this_thread::sleep_for(std::chrono::milliseconds(ms)); }
#define EXPECT(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); fflush(stdout); std::_Exit(1); } } while (0)

int main()
{
    SharedUnits u;
    // 190 and 190 of 256 do not go together
    std::atomic<int> second{0};
    u.take(190, 256);
    std::thread b([&] { u.take(190, 256); second = 1; });
    pause_ms(200);
    EXPECT(second == 0);
    u.give(190);
    b.join();
    EXPECT(second == 1);
    u.give(190);

    // one that wants nearly everything came before a small one that would fit: it is served first
    std::atomic<int> served{0}, big{0}, small{0};
    u.take(100, 256);
    std::thread large([&] { u.take(250, 256); big = ++served; pause_ms(50); u.give(250); });
    pause_ms(200);
    std::thread little([&] { u.take(10, 256); small = ++served; u.give(10); });
    pause_ms(200);
    EXPECT(served == 0);
    u.give(100);
    large.join();
    little.join();
    EXPECT(big == 1 && small == 2);

    // all of them together, and all units back at the end
    std::atomic<int> held{0}, most{0};
    std::vector<std::thread> threads;
    for (int i = 0; i < 8; ++i)
        threads.emplace_back([&, i] {
            for (int r = 0; r < 300; ++r) {
                const int want = 1 + (i * 37 + r * 11) % 256;
                u.take(want, 256);
                const int now = held += want;
                int seen = most;
                while (now > seen && !most.compare_exchange_weak(seen, now)) {}
                held -= want;
                u.give(want);
            }
        });
    for (std::thread &t : threads) t.join();
    EXPECT(most <= 256);
    u.take(256, 256);
    u.give(256);
    printf("ok\n");
    return 0;
}
"""


def test_units_are_never_more_than_the_device_has_and_are_given_in_turn(tmp_path):
    src, exe = tmp_path / "units.cpp", tmp_path / "units"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_2211_00839_amd", "csrc"), str(src),
                    "-o", str(exe)], check=True, timeout=60)
    res = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
